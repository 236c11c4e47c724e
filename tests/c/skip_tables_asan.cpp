// Driver of the host code that builds what the posterior kernels test and read
// (tests/test_asan_tables.py; built like plan_tables_asan.cpp, host only, with
// AddressSanitizer and UndefinedBehaviorSanitizer): the boxes along the nodes'
// principal axes, headers with their segments, probe operands, chunk records,
// super-tile centres and the skip depths, for ragged and square grids of every
// super-tile side, with and without the illumination projection, with the
// reference concentration inside and far off the grid.  Prints "skip tables
// asan ok" and returns 0 on success.
#include "hb_plan.cpp"

#include <cstdio>

namespace hb {
hipError_t launch_tikhonov_fp64(const double *, double *, float *, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_log_haar(const void *, int, const HaarArgs &, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_reference(const PosteriorArgs &, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_posterior(const PosteriorArgs &, bool, hipStream_t) { return hipErrorInvalidValue; }
hipError_t launch_recompose(int, const RecomposeArgs &, hipStream_t) { return hipErrorInvalidValue; }
hipError_t static_scratch(int, void **ptr) {
    *ptr = nullptr;
    return hipErrorInvalidValue;
}
}  // namespace hb

static int fail(const char *what, int a, int b) {
    std::fprintf(stderr, "skip tables asan: %s (%d, %d)\n", what, a, b);
    return 1;
}

// The three parts of a split value (slots 0, 1 and 3, or 2 for the norm).
static float joined(const uint16_t *operand, int lane) {
    const uint16_t *L = operand + (size_t)lane * (kSplitLaneBytes / 2);
    return (bf16_value(L[0]) + bf16_value(L[1])) + bf16_value(L[lane < 48 ? 3 : 2]);
}

static int check_tables(const hb_plan_desc_t &d, const std::vector<float> &table, int side) {
    const int nss = (d.grid_so2 + side - 1) / side, n_sup = (d.grid_thb + side - 1) / side * nss;
    const int stride = super_floats(side), cps = (side / 4) * (side / 4), slots = probe_slots(side);
    float origin[3], axes[9];
    grid_middle(table, n_sup, side, origin);
    principal_axes(table, n_sup, side, axes);
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            double dot = 0;
            for (int k = 0; k < 3; ++k) dot += (double)axes[3 * i + k] * (double)axes[3 * j + k];
            if (!(std::fabs(dot - (i == j)) < 1e-6)) return fail("axes not orthonormal", i, j);
        }
    const size_t boxes_at = (size_t)n_sup * kHdrFloats;
    std::vector<float> tests;
    std::vector<uint16_t> probes, records;
    build_test_tables(table, n_sup, nss, side, boxes_at, origin, axes, tests, probes);
    build_split_ops(table, n_sup, side, records, kChunkRecordBytes);
    if (tests.size() != boxes_at + (size_t)n_sup * cps * kBoxFloats ||
        probes.size() != ((size_t)n_sup * slots + 15) / 16 * (kSplitChunkBytes / 2) ||
        records.size() != (size_t)n_sup * cps * (kChunkRecordBytes / 2))
        return fail("table sizes", d.grid_thb, d.grid_so2);
    std::vector<char> taken((probes.size() / (kSplitChunkBytes / 2)) * 16, 0);   // probe slots in use
    for (int si = 0; si < n_sup; ++si) {
        const float *T = &table[(size_t)si * stride], *H = &tests[(size_t)si * kHdrFloats];
        int segment, np;
        std::memcpy(&segment, &H[14], sizeof(int));
        std::memcpy(&np, &T[14], sizeof(int));
        if (segment != (si / nss + si % nss) % kSegments) return fail("segment", si, segment);
        for (int k = 0; k < 3; ++k)
            if (H[8 + k] != T[k] || H[11 + k] != T[3 + k]) return fail("header centre", si, k);
        if (H[6] != T[6] || H[7] != T[7]) return fail("header concentrations", si, 0);
        // the distance between two centres is a float32 value
        const float *first = &table[0];
        for (int k = 6; k < 8; ++k)
            if ((double)(T[k] - first[k]) != (double)T[k] - (double)first[k]) return fail("centres not on a quantum", si, k);
        if (np < 1 || np > slots) return fail("probes of a super-tile", si, np);
        for (int i = 0; i < np; ++i) {
            const size_t at = (size_t)si * slots + i;
            const uint16_t *O = &probes[at / 16 * (kSplitChunkBytes / 2)];
            taken[at] = 1;
            double sq = 0;
            for (int k = 0; k < 3; ++k) {
                const double x = (((double)T[k] - (double)origin[k]) + (double)T[3 + k]) +
                                 (double)T[kSupHdr + i * kProbeFloats + k];
                const float got = joined(O, 16 * k + (int)(at % 16));
                if (got != (float)x) return fail("probe coordinate", si, i);
                sq += (double)got * (double)got;
            }
            if (joined(O, 48 + (int)(at % 16)) != (float)-sq) return fail("probe norm", si, i);
        }
        for (int c = 0; c < cps; ++c) {
            const float *C = T + kSupHdr + kMaxProbes * kProbeFloats + (size_t)c * kChunkFloats;
            const float *X = &tests[boxes_at + ((size_t)si * cps + c) * kBoxFloats];
            const uint16_t *R = &records[((size_t)si * cps + c) * (kChunkRecordBytes / 2)];
            float rows[16];
            std::memcpy(rows, R + kSplitChunkBytes / 2, sizeof(rows));
            for (int j = 0; j < kChunkNodes; ++j) {
                for (int k = 0; k < 4; ++k)
                    if (joined(R, 16 * k + j) != C[16 * k + j]) return fail("record operand", si, c);
                if (C[48 + j] == kPadLogit) continue;
                for (int r = 0; r < 3; ++r) {
                    // the node along the axis, and the rounding of that sum in FP64
                    double at = 0, size = 0;
                    for (int k = 0; k < 3; ++k) {
                        const double x = (((double)T[k] - (double)origin[k]) + (double)T[3 + k]) + (double)C[16 * k + j];
                        at += (double)axes[3 * r + k] * x;
                        size += std::fabs(x);
                    }
                    const double eps = 1e-14 * size;
                    if (!((double)X[r] <= at + eps && at - eps <= (double)X[3 + r])) return fail("box misses a node", si, c);
                    if (!(H[r] <= X[r] && X[3 + r] <= H[3 + r])) return fail("header box misses a chunk", si, c);
                }
                // the row's affine moments give the node's
                const float *Q = rows + 4 * (j / 4);
                const double hb = (double)Q[0] + (double)Q[1] * (j % 4), tol = 4e-7 * d.thb_max;
                if (!(std::fabs(hb - (double)C[64 + j]) <= tol && std::fabs((double)Q[2] - hb - (double)C[80 + j]) <= tol))
                    return fail("row moments", si, c);
            }
        }
    }
    // slots without a probe never win
    for (size_t at = 0; at < taken.size(); ++at)
        if (!taken[at] && joined(&probes[at / 16 * (kSplitChunkBytes / 2)], 48 + (int)(at % 16)) != kPadLogit)
            return fail("empty probe slot", (int)at, 0);
    return 0;
}

int main() {
    ForwardModel fm;
    fm.n = 9;
    fm.L = 0.1;
    for (int j = 0; j < fm.n; ++j) {
        fm.ehb.push_back(0.02 + 0.01 * j);
        fm.eox.push_back(0.05 - 0.004 * j);
    }
    for (int k = 0; k < 3; ++k) {
        double s = 0;
        std::vector<double> row;
        for (int j = 0; j < fm.n; ++j) row.push_back(std::exp(-0.5 * (j - 3.0 * k - 1.0) * (j - 3.0 * k - 1.0)));
        for (double v : row) s += v;
        for (double v : row) fm.resp.push_back(v / s);
    }
    const int grids[][2] = {{1, 1}, {3, 5}, {16, 16}, {33, 7}, {40, 40}, {64, 45}, {100, 37}, {128, 128}, {170, 200},
                            {256, 256}, {300, 17}};
    for (const auto &g : grids)
        for (int illum = 0; illum < 2; ++illum)
            for (double ref : {70.0, 0.0, 900.0}) {
                hb_plan_desc_t d;
                hb_plan_desc_default(&d);
                d.grid_thb = g[0];
                d.grid_so2 = g[1];
                d.illumination = illum;
                if (ref != 70.0) {
                    d.thb_min = 100.0;
                    d.thb_max = 100.5;
                }
                const int side = super_side(d.grid_thb, d.grid_so2);
                double mu_ref[3], direct_index;
                fm.mu(0.4 * ref, 0.6 * ref, mu_ref);
                std::vector<float> table, lo;
                build_supers(d, fm, mu_ref, ref == 70.0 ? 40.0 : 4.0e4, side, table, lo, direct_index);
                const int r = check_tables(d, table, side);
                if (r) return r;
            }
    // Depths of a plan: the first lies between its floor and the a-priori
    // threshold, and what is certified moves a mean by less than the bound; a split
    // grid and exact skipping have one depth.
    for (int grid : {8, 64, 256, 1024})
        for (double tol : {1e-12, 1e-9, 1e-6, 1e-4, 1e-2, 1.0, 100.0})
            for (int split : {1, 4}) {
                hb_plan_s p;
                hb_plan_desc_default(&p.desc);
                p.desc.posterior_tolerance = tol;
                p.n_nodes = (long long)grid * grid;
                set_split(&p, split);
                if (p.info.grid_split != split || !(p.depth0 >= kMinSkipLog2 && p.depth0 <= p.skip_log2))
                    return fail("first depth", grid, split);
                if (split > 1 && p.depth0 != p.skip_log2) return fail("depth of a split grid", grid, split);
                if (split == 1 && p.info.skip_bound > 0 && !(std::exp2((double)p.cert_log2) * p.desc.thb_max < p.info.skip_bound))
                    return fail("certified ratio", grid, split);
                p.desc.posterior_tolerance = 0.0;
                set_split(&p, split);
                if (p.depth0 != kExactSkipLog2 || p.info.skip_bound != 0.0) return fail("exact depth", grid, split);
            }
    std::printf("skip tables asan ok\n");
    return 0;
}
