// Host-only setup pieces: CSR validation, transposed index, row schedule.
// Nothing here touches the GPU, so these entry points can be checked on a
// machine without one.
#include "sdnn_internal.h"

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <numeric>
#include <vector>

static thread_local char g_err[512] = "";

void sdnn_set_global_error(const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof g_err, fmt, ap);
    va_end(ap);
}
const char *sdnn_global_error() { return g_err; }

extern "C" int sdnn_check_csr(int32_t n_out, int32_t n_in, const int32_t *row_ptr,
                              const int32_t *col_idx)
{
    if (n_out < 0 || n_in < 0) { sdnn_set_global_error("negative matrix size"); return SDNN_EINVAL; }
    if (!row_ptr) { sdnn_set_global_error("row_ptr is NULL"); return SDNN_EINVAL; }
    if (row_ptr[0] != 0) { sdnn_set_global_error("row_ptr[0] != 0"); return SDNN_EINVAL; }
    for (int32_t j = 0; j < n_out; ++j)
        if (row_ptr[j + 1] < row_ptr[j]) {
            sdnn_set_global_error("row_ptr decreases at row %d", j);
            return SDNN_EINVAL;
        }
    if (row_ptr[n_out] > 0 && !col_idx) { sdnn_set_global_error("col_idx is NULL"); return SDNN_EINVAL; }
    for (int32_t j = 0; j < n_out; ++j)
        for (int32_t p = row_ptr[j]; p < row_ptr[j + 1]; ++p) {
            if (col_idx[p] < 0 || col_idx[p] >= n_in) {
                sdnn_set_global_error("column %d out of range in row %d", col_idx[p], j);
                return SDNN_EINVAL;
            }
            if (p > row_ptr[j] && col_idx[p] <= col_idx[p - 1]) {
                sdnn_set_global_error("columns of row %d are not strictly ascending", j);
                return SDNN_EINVAL;
            }
        }
    return SDNN_OK;
}

// Counting sort by column; visiting the rows in ascending order makes every
// transposed row list its source rows in ascending order, which fixes the
// summation order of the backward product.
extern "C" int sdnn_transpose_pattern(int32_t n_out, int32_t n_in, const int32_t *row_ptr,
                                      const int32_t *col_idx, int32_t *t_row_ptr,
                                      int32_t *t_row_idx, int32_t *t_perm)
{
    if (!row_ptr || !t_row_ptr) { sdnn_set_global_error("NULL pointer"); return SDNN_EINVAL; }
    const int32_t nnz = row_ptr[n_out];
    if (nnz > 0 && (!col_idx || !t_row_idx || !t_perm)) {
        sdnn_set_global_error("NULL pointer");
        return SDNN_EINVAL;
    }
    std::fill(t_row_ptr, t_row_ptr + n_in + 1, 0);
    for (int32_t p = 0; p < nnz; ++p) t_row_ptr[col_idx[p] + 1]++;
    for (int32_t i = 0; i < n_in; ++i) t_row_ptr[i + 1] += t_row_ptr[i];
    try {
        std::vector<int32_t> cursor(t_row_ptr, t_row_ptr + n_in);
        for (int32_t j = 0; j < n_out; ++j)
            for (int32_t p = row_ptr[j]; p < row_ptr[j + 1]; ++p) {
                const int32_t q = cursor[col_idx[p]]++;
                t_row_idx[q] = j;
                t_perm[q] = p;
            }
    } catch (...) { // nothing may cross the C boundary
        sdnn_set_global_error("host allocation failed");
        return SDNN_ENOMEM;
    }
    return SDNN_OK;
}

extern "C" int sdnn_row_schedule(int32_t n_rows, const int32_t *row_ptr, int32_t *order)
{
    if (n_rows < 0 || !row_ptr || (n_rows > 0 && !order)) {
        sdnn_set_global_error("NULL pointer or negative size");
        return SDNN_EINVAL;
    }
    int32_t longest = 0;
    for (int32_t r = 0; r < n_rows; ++r) {
        if (row_ptr[r + 1] < row_ptr[r]) {
            sdnn_set_global_error("row_ptr decreases at row %d", r);
            return SDNN_EINVAL;
        }
        longest = std::max(longest, row_ptr[r + 1] - row_ptr[r]);
    }
    try {
        if (longest / 16 > n_rows) { // a few long rows: counting would take more memory than the rows do
            std::iota(order, order + n_rows, 0);
            std::stable_sort(order, order + n_rows, [&](int32_t a, int32_t b) { return row_ptr[a + 1] - row_ptr[a] > row_ptr[b + 1] - row_ptr[b]; });
            return SDNN_OK;
        }
        // counting sort by decreasing length, stable
        std::vector<int32_t> at((size_t)longest + 2, 0); // at[longest - len]: the next place of a row of that length
        for (int32_t r = 0; r < n_rows; ++r) at[(size_t)(longest - (row_ptr[r + 1] - row_ptr[r])) + 1]++;
        for (int32_t k = 0; k <= longest; ++k) at[(size_t)k + 1] += at[(size_t)k];
        for (int32_t r = 0; r < n_rows; ++r) order[at[(size_t)(longest - (row_ptr[r + 1] - row_ptr[r]))]++] = r;
    } catch (...) {
        sdnn_set_global_error("host allocation failed");
        return SDNN_ENOMEM;
    }
    return SDNN_OK;
}

// Greedy clustering of rows by shared columns, one pass over the entries.  Every column remembers
// the cluster of the last row that used it; a row joins the open cluster that most of its columns
// point at (if at least a quarter of them do), otherwise it opens a new cluster.  Clusters are
// closed at max_cluster_rows rows.  The result lists the rows cluster by cluster, clusters by
// decreasing longest row (so the longest-first dealing of the row schedule survives between
// clusters), rows inside a cluster by decreasing length, ties in arrival order.
extern "C" int sdnn_cluster_rows(int32_t n_rows, int32_t n_cols, const int32_t *row_ptr, const int32_t *col_idx,
                                 int32_t max_cluster_rows, int32_t *order, int32_t *cluster_of)
{
    if (n_rows < 0 || n_cols < 0 || !row_ptr || (n_rows > 0 && !order) || max_cluster_rows < 1) {
        sdnn_set_global_error("NULL pointer or bad size");
        return SDNN_EINVAL;
    }
    if (row_ptr[n_rows] > 0 && !col_idx) { sdnn_set_global_error("col_idx is NULL"); return SDNN_EINVAL; }
    try {
        std::vector<int32_t> last((size_t)n_cols, -1);  // column -> cluster of the last row that used it
        std::vector<int32_t> size, longest;             // per cluster
        std::vector<int32_t> votes, touched;            // scratch: votes per cluster of the current row
        std::vector<int32_t> member((size_t)n_rows, -1);
        for (int32_t j = 0; j < n_rows; ++j) {
            const int32_t beg = row_ptr[j], end = row_ptr[j + 1], len = end - beg;
            int32_t best = -1, best_votes = 0;
            touched.clear();
            for (int32_t p = beg; p < end; ++p) {
                const int32_t c = last[col_idx[p]];
                if (c < 0 || size[c] >= max_cluster_rows) continue;
                if (votes[c]++ == 0) touched.push_back(c);
                if (votes[c] > best_votes || (votes[c] == best_votes && c < best)) { best_votes = votes[c]; best = c; }
            }
            for (int32_t c : touched) votes[c] = 0;
            if (best < 0 || 4 * best_votes < len) { // nothing worth joining: a cluster of its own
                best = (int32_t)size.size();
                size.push_back(0);
                longest.push_back(0);
                votes.push_back(0);
            }
            member[j] = best;
            size[best]++;
            longest[best] = std::max(longest[best], len);
            for (int32_t p = beg; p < end; ++p) last[col_idx[p]] = best;
        }
        const int32_t n_clusters = (int32_t)size.size();
        std::vector<int32_t> corder((size_t)n_clusters);
        std::iota(corder.begin(), corder.end(), 0);
        std::stable_sort(corder.begin(), corder.end(), [&](int32_t a, int32_t b) { return longest[a] > longest[b]; });
        std::vector<int32_t> rank((size_t)n_clusters);
        for (int32_t k = 0; k < n_clusters; ++k) rank[corder[k]] = k;
        std::iota(order, order + n_rows, 0);
        std::stable_sort(order, order + n_rows, [&](int32_t a, int32_t b) {
            if (rank[member[a]] != rank[member[b]]) return rank[member[a]] < rank[member[b]];
            return row_ptr[a + 1] - row_ptr[a] > row_ptr[b + 1] - row_ptr[b];
        });
        if (cluster_of)
            for (int32_t j = 0; j < n_rows; ++j) cluster_of[j] = rank[member[j]];
    } catch (...) {
        sdnn_set_global_error("host allocation failed");
        return SDNN_ENOMEM;
    }
    return SDNN_OK;
}

// Deals a row order out to the 8 XCDs.  Workgroups take 4 consecutive rows of the schedule and
// workgroup ids go to the XCDs round-robin, so rows 32q + 4x .. 32q + 4x + 3 of the schedule run on
// XCD x.  The rows of `order` (neighbours share columns) are cut into 8 contiguous stretches of about
// equal numbers of entries, and stretch x fills the places of XCD x: neighbours then run on one XCD
// (one L2) and, four at a time, on one CU at about the same moment.  When the stretches differ in
// length the places left over at the end are filled from the remaining stretches in turn.
extern "C" int sdnn_deal_rows_to_xcds(int32_t n_rows, const int32_t *row_ptr, const int32_t *order, int32_t *dealt)
{
    if (n_rows < 0 || !row_ptr || (n_rows > 0 && (!order || !dealt))) {
        sdnn_set_global_error("NULL pointer or negative size");
        return SDNN_EINVAL;
    }
    const int X = 8, G = 4;
    try {
        // cut points by entries (+1 per row so that empty rows count too)
        int64_t total = 0;
        for (int32_t r = 0; r < n_rows; ++r) total += row_ptr[order[r] + 1] - row_ptr[order[r]] + 1;
        std::vector<int32_t> cut(X + 1, n_rows);
        cut[0] = 0;
        int64_t acc = 0;
        int x = 1;
        for (int32_t r = 0; r < n_rows && x < X; ++r) {
            acc += row_ptr[order[r] + 1] - row_ptr[order[r]] + 1;
            while (x < X && acc * X >= total * x) cut[x++] = r + 1;
        }
        std::vector<int32_t> next(cut.begin(), cut.begin() + X); // read position of every stretch
        for (int32_t pos = 0; pos < n_rows; ++pos) {
            int xcd = (pos / G) % X;
            for (int t = 0; t < X && next[xcd] >= cut[xcd + 1]; ++t) xcd = (xcd + 1) % X; // stretch used up: the next one
            dealt[pos] = order[next[xcd]++];
        }
    } catch (...) {
        sdnn_set_global_error("host allocation failed");
        return SDNN_ENOMEM;
    }
    return SDNN_OK;
}

void sdnn_pan_geometry(const sdnn_layer &y, const PanLayer *below, PanLayer &g)
{
    auto cut = [](int32_t n, int32_t &parts, int32_t &each) {
        parts = (n + PAN_POS - 1) / PAN_POS;
        each = ((n + parts - 1) / parts + 63) & ~63;
    };
    if (below) { // a panel is what one range of the layer below has written
        g.n_panels = below->n_ranges;
        g.panel_cols = below->range_rows;
        g.panel = below->range;
        g.in_pos = below->out_pos;
    } else {
        cut(y.n_in, g.n_panels, g.panel_cols);
        g.panel = g.panel_cols;
        g.in_pos = y.n_in;
    }
    cut(y.n_out, g.n_ranges, g.range_rows);
    g.nb = (g.range_rows + 64 * PAN_WAVES - 1) / (64 * PAN_WAVES);
    g.range = 64 * PAN_WAVES * g.nb;
    g.out_pos = g.n_ranges * g.range;
    const size_t streams = (size_t)g.n_ranges * PAN_WAVES;
    g.halves = (size_t)(PAN_SLOTS * (double)y.row_ptr[y.n_out] / 512.0) + streams * ((size_t)g.n_panels * (size_t)(g.nb + 8) / 8 + 7) + 4;
    g.halves = (g.halves + 3) & ~(size_t)3;
}

// How many of a row's columns are below `bound`: four at a time, without branches on them.
static int32_t entries_below(const int32_t *c, int32_t len, int32_t bound)
{
    typedef int32_t four __attribute__((vector_size(16)));
    const four bounds = {bound, bound, bound, bound};
    four sum = {0, 0, 0, 0};
    int32_t e = 0;
    for (; e + 4 <= len; e += 4) {
        four v;
        std::memcpy(&v, c + e, sizeof v);
        sum -= v < bounds; // -1 where it holds
    }
    int32_t n = sum[0] + sum[1] + sum[2] + sum[3];
    for (; e < len; ++e) n += c[e] < bound;
    return n;
}

// A wavefront's lanes walk their rows in step, so a block of 64 rows costs as many slots in a panel as its fullest row has
// entries there.  The rows of a range are halved, again and again, at the median of the panel in which their counts spread most,
// until 64 are left: their counts are then about equal in every panel (32 entries per row over four panels: 1.10 slots per entry,
// against 1.76 for rows as they come).
void sdnn_pan_layout(const sdnn_layer &y, const PanLayer &g, PanLayout &out)
{
    const int32_t P = g.n_panels, S = (P + 3) & ~3, nb = g.nb; // a row's counts: P, and zeros up to a multiple of four
    std::vector<int32_t> count((size_t)y.n_out * S, 0), order, of_row, rows_of_count, second;
    std::vector<int64_t> per_panel((size_t)P, 0);
    for (int32_t r = 0; r < y.n_out; ++r) {
        const int32_t *const c = y.col_idx + y.row_ptr[r], len = y.row_ptr[r + 1] - y.row_ptr[r];
        int32_t before = 0;
        for (int32_t p = 0; p < P; ++p) {
            int32_t below = len; // entries of this panel and those before it
            if (p < P - 1) { // columns ascend; of short rows all entries are looked at, the same number for every panel and row
                const int32_t from = len > 128 ? before : 0;
                below = from + entries_below(c + from, len - from, (p + 1) * g.panel_cols);
            }
            count[(size_t)r * S + p] = below - before;
            per_panel[(size_t)p] += below - before;
            before = below;
        }
    }
    out.fullest = *std::max_element(per_panel.begin(), per_panel.end());
    out.rows.assign((size_t)g.out_pos, -1);
    out.pos.assign((size_t)y.n_out, 0);
    out.seg.assign((size_t)g.n_ranges * PAN_WAVES * (P + 1), 0);
    out.slot.assign((size_t)g.n_ranges * PAN_WAVES * P * (nb + 1), 0);
    out.ends.clear();
    out.depth = 0;
    int32_t at = 0; // slots so far
    struct Block { int32_t first, n; int64_t slots; };
    std::vector<Block> blocks;
    std::vector<int32_t> members[PAN_WAVES];
    std::vector<int32_t> depth; // [block][panel]
    for (int32_t q = 0; q < g.n_ranges; ++q) {
        const int32_t r0 = std::min(y.n_out, q * g.range_rows), r1 = std::min(y.n_out, r0 + g.range_rows);
        order.resize((size_t)(r1 - r0));
        std::iota(order.begin(), order.end(), r0);
        blocks.clear();
        std::vector<std::pair<int32_t, int32_t>> todo(1, {0, r1 - r0});
        while (!todo.empty()) {
            const int32_t a = todo.back().first, b = todo.back().second;
            todo.pop_back();
            if (b - a <= 64) {
                if (b > a) blocks.push_back({a, b - a, 0});
                continue;
            }
            int32_t by = 0, sum[PAN_MAX] = {};   // (at most PAN_POS rows of at most PAN_POS entries)
            double sq[PAN_MAX] = {}, most = -1;
            for (int32_t p0 = 0; p0 < S; p0 += 4) {
                int32_t s4[4] = {};
                double q4[4] = {};
                for (int32_t k = a; k < b; ++k) {
                    const int32_t *c = count.data() + (size_t)order[(size_t)k] * S + p0;
                    for (int i = 0; i < 4; ++i) {
                        s4[i] += c[i];
                        q4[i] += (double)c[i] * c[i];
                    }
                }
                std::copy_n(s4, 4, sum + p0);
                std::copy_n(q4, 4, sq + p0);
            }
            for (int32_t p = 0; p < P; ++p) {
                const double spread = sq[p] - (double)sum[p] * (double)sum[p] / (b - a);
                if (spread > most) { most = spread; by = p; }
            }
            // the fullest rows first, ties by row: `order` ascends in every part, so a pass that keeps it that way does both
            const int32_t m = a + ((b - a + 63) / 64 + 1) / 2 * 64;
            of_row.resize((size_t)(b - a));
            int32_t fullest = 0;
            for (int32_t k = a; k < b; ++k) {
                const int32_t c = count[(size_t)order[(size_t)k] * S + by];
                of_row[(size_t)(k - a)] = c;
                fullest = std::max(fullest, c);
            }
            rows_of_count.assign((size_t)fullest + 1, 0);
            for (int32_t k = 0; k < b - a; ++k) rows_of_count[(size_t)of_row[(size_t)k]]++;
            int32_t median = fullest, left = m - a; // rows of more than `median` entries go first, and `left` of just so many
            while (rows_of_count[(size_t)median] < left) left -= rows_of_count[(size_t)median--];
            second.resize((size_t)(b - a));
            int32_t n0 = a, n1 = 0;
            for (int32_t k = a; k < b; ++k) {
                const int32_t c = of_row[(size_t)(k - a)], row = order[(size_t)k];
                const int32_t tie = c == median && left > 0, first = (c > median) | tie;
                left -= tie;
                order[(size_t)n0] = row; // (both are written, one counts)
                second[(size_t)n1] = row;
                n0 += first;
                n1 += !first;
            }
            std::copy_n(second.begin(), n1, order.begin() + m);
            todo.push_back({m, b});
            todo.push_back({a, m});
        }
        depth.assign(blocks.size() * P, 1); // every block has a slot in every panel, after which the next one's turn follows
        for (size_t k = 0; k < blocks.size(); ++k)
            for (int32_t p = 0; p < P; ++p) {
                int32_t &d = depth[k * P + p];
                for (int32_t i = 0; i < blocks[k].n; ++i) d = std::max(d, count[(size_t)order[(size_t)(blocks[k].first + i)] * S + p]);
                blocks[k].slots += d;
            }
        // dealt to the wavefronts, the deepest first, each to the one with the fewest slots so far
        std::vector<int32_t> by_depth(blocks.size());
        std::iota(by_depth.begin(), by_depth.end(), 0);
        std::stable_sort(by_depth.begin(), by_depth.end(), [&](int32_t u, int32_t v) { return blocks[u].slots > blocks[v].slots; });
        int64_t load[PAN_WAVES] = {};
        for (auto &m : members) m.clear();
        for (int32_t k : by_depth) {
            int w = -1;
            for (int i = 0; i < PAN_WAVES; ++i)
                if ((int32_t)members[i].size() < nb && (w < 0 || load[i] < load[w])) w = i;
            load[w] += blocks[k].slots;
            members[w].push_back(k);
        }
        std::vector<int64_t> deepest((size_t)P, 0);
        for (int w = 0; w < PAN_WAVES; ++w) {
            at = (at + 31) & ~31; // a multiple of four halves
            for (size_t j = 0; j < members[w].size(); ++j) {
                const Block &b = blocks[members[w][j]];
                for (int32_t i = 0; i < b.n; ++i) {
                    const int32_t local = 64 * (PAN_WAVES * (int32_t)j + w) + i, row = order[(size_t)(b.first + i)];
                    out.rows[(size_t)(q * g.range + local)] = row;
                    out.pos[(size_t)row] = q * g.range + local;
                }
            }
            int32_t *seg = out.seg.data() + (size_t)(q * PAN_WAVES + w) * (P + 1);
            for (int32_t p = 0; p < P; ++p) {
                const int32_t from = at;
                int32_t *slot = out.slot.data() + ((size_t)(q * PAN_WAVES + w) * P + p) * (nb + 1);
                seg[p] = at / 8;
                out.ends.resize((size_t)at / 8 + 1, 0);
                for (int32_t j = 0; j < nb; ++j) {
                    slot[j] = at;
                    if (j >= (int32_t)members[w].size()) continue;
                    at += depth[(size_t)members[w][j] * P + p];
                    out.ends.resize((size_t)(at - 1) / 8 + 1, 0);
                    if (j + 1 < (int32_t)members[w].size()) out.ends[(size_t)(at - 1) / 8] |= (uint8_t)(1u << ((at - 1) & 7));
                }
                if (members[w].empty()) at += 1; // a wavefront without rows takes part in the barriers
                const int32_t used = std::max<int32_t>(1, (int32_t)members[w].size());
                at = p < P - 1 ? (at + 7) & ~7 : (at + 15) & ~15; // a whole half; at the end an even number of them
                for (int32_t j = used; j <= nb; ++j) slot[j] = at; // the last block's slots are filled up to a batch
                deepest[(size_t)p] = std::max<int64_t>(deepest[(size_t)p], at - from);
            }
            seg[P] = at / 8;
        }
        double d = 0;
        for (int64_t v : deepest) d += (double)v;
        out.depth = std::max(out.depth, d);
    }
    out.ends.resize(((size_t)at + 31) / 32 * 4, 0);
}

extern "C" const char *sdnn_version(void) { return "sdnn 0.1 (gfx950)"; }
