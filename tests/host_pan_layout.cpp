// The layout of the forward in panels (sdnn_pan_geometry, sdnn_pan_layout), walked on the host as the kernels write and read
// it: built and run by tests/test_pan_layout.py with g++ under AddressSanitizer and UBSan.
// Arguments: the widths of the layers; links per row are drawn from 0 to 40.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <set>
#include <vector>

#include "../paper_2104_11805_amd/csrc/sdnn_internal.h"

static uint32_t state = 4711u;
static uint32_t rnd() { state = state * 1664525u + 1013904223u; return state >> 8; }
#define CHECK(x) do { if (!(x)) { std::printf("failed: %s (layer %d)\n", #x, l); return 1; } } while (0)

int main(int argc, char **argv)
{
    std::vector<int32_t> below_pos;
    std::vector<PanLayer> geo((size_t)argc);
    for (int l = 0; l + 2 < argc; ++l) {
        const int n_in = atoi(argv[l + 1]), n_out = atoi(argv[l + 2]);
        std::vector<int32_t> row_ptr(n_out + 1, 0), col;
        for (int r = 0; r < n_out; ++r) {
            std::set<int32_t> c;
            for (int k = (int)(rnd() % 41); k > 0; --k) c.insert((int32_t)(rnd() % n_in));
            col.insert(col.end(), c.begin(), c.end());
            row_ptr[r + 1] = (int32_t)col.size();
        }
        const sdnn_layer y = {n_out, n_in, row_ptr.data(), col.data(), nullptr, nullptr};
        PanLayer &g = geo[l];
        sdnn_pan_geometry(y, l > 0 ? &geo[l - 1] : nullptr, g);
        PanLayout out;
        sdnn_pan_layout(y, g, out);
        CHECK(g.panel <= PAN_POS && g.range <= PAN_POS && g.panel_cols <= g.panel && g.panel % 64 == 0);
        CHECK(g.n_panels * (int64_t)g.panel_cols >= n_in && g.n_ranges * (int64_t)g.range_rows >= n_out);
        CHECK(out.ends.size() % 4 == 0 && (int)out.rows.size() == g.out_pos && out.ends.size() <= g.halves);
        // every row has a place of its own, inside the range that holds it
        for (int r = 0; r < n_out; ++r) CHECK(out.rows[out.pos[r]] == r && out.pos[r] / g.range == r / g.range_rows);
        int placed = 0;
        for (int32_t r : out.rows) placed += r >= 0;
        CHECK(placed == n_out);
        // the slots, as k_pan_fill writes them: entry, or -1 for one past a row's entries in the panel
        const size_t n_slots = 8 * out.ends.size();
        std::vector<int32_t> entry(n_slots * 64, -2);
        for (int q = 0; q < g.n_ranges; ++q)
            for (int w = 0; w < PAN_WAVES; ++w)
                for (int p = 0; p < g.n_panels; ++p)
                    for (int j = 0; j < g.nb; ++j) {
                        const int32_t *slot = out.slot.data() + ((size_t)(q * PAN_WAVES + w) * g.n_panels + p) * (g.nb + 1) + j;
                        for (int lane = 0; lane < 64; ++lane) {
                            const int row = out.rows[q * g.range + 64 * (PAN_WAVES * j + w) + lane];
                            std::vector<int32_t> mine;
                            for (int e = row < 0 ? 0 : row_ptr[row]; row >= 0 && e < row_ptr[row + 1]; ++e)
                                if (col[e] / g.panel_cols == p) mine.push_back(e);
                            CHECK((int)mine.size() <= slot[1] - slot[0]);
                            for (int s = slot[0]; s < slot[1]; ++s) {
                                CHECK(s >= 0 && (size_t)s < n_slots && entry[(size_t)s * 64 + lane] == -2); // no slot twice
                                entry[(size_t)s * 64 + lane] = s - slot[0] < (int)mine.size() ? mine[s - slot[0]] : -1;
                            }
                        }
                    }
        // and as k_fwd_pan reads them: every row meets its entries in storage order, each while its panel is in LDS
        std::vector<int32_t> next(row_ptr.begin(), row_ptr.end() - 1);
        for (int q = 0; q < g.n_ranges; ++q)
            for (int w = 0; w < PAN_WAVES; ++w) {
                const int32_t *seg = out.seg.data() + (size_t)(q * PAN_WAVES + w) * (g.n_panels + 1);
                CHECK(seg[0] % 4 == 0 && (seg[g.n_panels] - seg[0]) % 2 == 0);
                for (int p = 0; p < g.n_panels; ++p) {
                    CHECK(seg[p + 1] > seg[p]); // every wavefront takes part in every panel's barriers
                    int j = 0;
                    for (int s = 8 * seg[p]; s < 8 * seg[p + 1]; ++s) {
                        for (int lane = 0; lane < 64; ++lane) {
                            const int32_t e = entry[(size_t)s * 64 + lane];
                            CHECK(e != -2);
                            if (e < 0) continue;
                            CHECK(j < g.nb);
                            const int row = out.rows[q * g.range + 64 * (PAN_WAVES * j + w) + lane];
                            CHECK(row >= 0 && next[row] == e && e < row_ptr[row + 1] && col[e] / g.panel_cols == p);
                            const int at = l > 0 ? below_pos[col[e]] : col[e];
                            CHECK(at >= p * g.panel && at < (p + 1) * g.panel && at < g.in_pos);
                            next[row] = e + 1;
                        }
                        if (out.ends[(size_t)s / 8] >> (s & 7) & 1) ++j;
                    }
                    CHECK(j < g.nb); // the sums that k_fwd_pan reaches by index
                }
            }
        for (int r = 0; r < n_out; ++r) CHECK(next[r] == row_ptr[r + 1]);
        below_pos = out.pos;
    }
    std::puts("pan layout: ok");
    return 0;
}
