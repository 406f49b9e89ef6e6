// Prints what the launch rules (csrc/launch.h) answer to the questions on standard input, one line each.  Built and
// asked by tests/test_launch_shape.py.
#include <cstdio>
#include <cstring>
#include <vector>

#include "launch.h"

int main() {
    char what[16];
    while (std::scanf("%15s", what) == 1) {
        if (!std::strcmp(what, "lds")) {              // lds kind few form cap
            int kind, few, form, cap;
            if (std::scanf("%d %d %d %d", &kind, &few, &form, &cap) != 4) return 1;
            const size_t own = static_lds(kind, few != 0, form);
            std::printf("%zu %zu\n", own, lds_for_workgroups_per_cu(cap, own));
        } else if (!std::strcmp(what, "have")) {      // have: what this build's tiles allow
            std::printf("%d %d %d\n", HAVE_PAIRS, HAVE_FEW, HAVE_PIECES);
        } else if (!std::strcmp(what, "on_lines")) {  // on_lines kind dtype reduced tiles segments off_lines
            LaunchWork w{};
            int reduced;
            if (std::scanf("%d %d %d %d %d %lf", &w.kind, &w.dtype, &reduced, &w.tiles, &w.segments, &w.off_lines) != 6) return 1;
            w.P = 3;
            w.reduced = reduced != 0;
            std::printf("%d\n", launch_shape(LaunchSettings{}, w, 256).on_lines);
        } else if (!std::strcmp(what, "through")) {   // through kind dtype tiles off_lines ragged segments
            LaunchWork w{};
            if (std::scanf("%d %d %d %lf %lf %d", &w.kind, &w.dtype, &w.tiles, &w.off_lines, &w.ragged, &w.segments) != 6) return 1;
            w.P = 8;
            std::printf("%d\n", launch_shape(LaunchSettings{}, w, 256).through);
        } else if (!std::strcmp(what, "cuts")) {      // cuts line L {n merged weights}...: tensor, begin and end of every tile's shares
            int line, L;
            if (std::scanf("%d %d", &line, &L) != 2) return 1;
            std::vector<uint64_t> n(static_cast<size_t>(L)), weights(static_cast<size_t>(L));
            std::vector<uint8_t> merged(static_cast<size_t>(L));
            for (size_t i = 0; i < n.size(); ++i) {
                unsigned long long elems, address;
                int m;
                if (std::scanf("%llu %d %llu", &elems, &m, &address) != 3) return 1;
                n[i] = elems;
                merged[i] = static_cast<uint8_t>(m);
                weights[i] = address;
            }
            HostTables h;
            if (mgwfbp_build_tables(n.data(), L, merged.data(), h) != MGWFBP_OK) return 1;
            for (size_t t = 0; t < h.tiles.size(); ++t) {
                const TileHdr& x = h.tiles[t];
                const int64_t base = static_cast<int64_t>(t) * TILE;
                auto early = [&](const TileHdr& y) { return starts_early(y.first_start, line_shift(weights[static_cast<size_t>(y.layer0)], y.first_start, line)); };
                const int64_t end = x.valid - (x.flags & TILE_GOES_ON ? early(h.tiles[t + 1]) : 0);
                for (int j = 0; j < x.nseg; ++j) {
                    const size_t q = static_cast<size_t>(x.seg0 + j);
                    const int64_t start = static_cast<int64_t>(h.seg_off[q]) - base, own = start + static_cast<int64_t>(h.seg_n[q]);
                    const int64_t lo = start < 0 ? -early(x) : start, hi = own < end ? own : end;
                    std::printf("%d %lld %lld ", h.seg_layer[q], static_cast<long long>(lo - start), static_cast<long long>(hi - start));
                }
            }
            std::printf("\n");
        } else if (!std::strcmp(what, "shape")) {     // shape <work> <settings> n_cu
            LaunchWork w{};
            LaunchSettings set;
            int reduced, n_cu;
            long long resident_bytes;
            if (std::scanf("%d %d %d %d %lf %lf %d %lf %d", &w.kind, &w.dtype, &w.P, &w.tiles, &w.ragged, &w.off_lines, &reduced,
                           &w.resident, &w.segments) != 9) return 1;
            if (std::scanf("%d %d %d %d %d %d %lld %d", &set.blocks_per_cu, &set.xcd_contiguous, &set.tiles_per_wg, &set.wg_per_cu,
                           &set.step_vecs, &set.burst_tiles, &resident_bytes, &n_cu) != 8) return 1;
            w.reduced = reduced != 0;
            set.resident_bytes = static_cast<uint64_t>(resident_bytes);
            const LaunchShape s = launch_shape(set, w, n_cu);
            std::printf("%d %d %d %d %d %d %d %d %d %d\n", s.tiles_per_wg, s.units, s.grid, s.xcd_contiguous, s.run_log2, s.may_be_few,
                        s.form, s.wgs_per_cu, s.rolling, s.in_pieces);
        } else if (!std::strcmp(what, "forms")) {     // forms P dtype reduced L {n merged}...: launches over all of a model, each kind's form,
                                                      // on_lines, through, may_be_few and run_log2
            LaunchWork w{};
            int reduced, L;
            if (std::scanf("%d %d %d %d", &w.P, &w.dtype, &reduced, &L) != 4) return 1;
            std::vector<uint64_t> n(static_cast<size_t>(L));
            std::vector<uint8_t> merged(static_cast<size_t>(L));
            for (size_t i = 0; i < n.size(); ++i) {
                unsigned long long elems;
                int m;
                if (std::scanf("%llu %d", &elems, &m) != 2) return 1;
                n[i] = elems;
                merged[i] = static_cast<uint8_t>(m);
            }
            HostTables h;
            if (mgwfbp_build_tables(n.data(), L, merged.data(), h) != MGWFBP_OK) return 1;
            w.reduced = reduced != 0;
            w.tiles = static_cast<int32_t>(h.tiles.size());
            w.segments = static_cast<int32_t>(h.seg_layer.size());
            const LaunchShares shares = shares_of(h, 0, w.segments, w.tiles);
            w.ragged = shares.ragged;
            w.off_lines = shares.off_lines;
            for (w.kind = K_PACK; w.kind <= K_DIRECT; ++w.kind) {
                const LaunchShape s = launch_shape(LaunchSettings{}, w, 256);
                std::printf("%d %d %d %d %d ", s.form, s.on_lines, s.through, s.may_be_few, s.run_log2);
            }
            std::printf("\n");
        } else if (!std::strcmp(what, "shares")) {    // shares L {n merged}... g0 g1: of the launch over groups [g0, g1)
            int L, g0, g1;
            if (std::scanf("%d", &L) != 1) return 1;
            std::vector<uint64_t> n(static_cast<size_t>(L));
            std::vector<uint8_t> merged(static_cast<size_t>(L));
            for (size_t i = 0; i < n.size(); ++i) {
                unsigned long long elems;
                int m;
                if (std::scanf("%llu %d", &elems, &m) != 2) return 1;
                n[i] = elems;
                merged[i] = static_cast<uint8_t>(m);
            }
            HostTables h;
            if (std::scanf("%d %d", &g0, &g1) != 2 || mgwfbp_build_tables(n.data(), L, merged.data(), h) != MGWFBP_OK) return 1;
            const size_t a = static_cast<size_t>(g0), b = static_cast<size_t>(g1 < 0 ? h.G : g1);
            const int32_t tiles = h.group_tile[b] - h.group_tile[a];
            const LaunchShares s = shares_of(h, h.group_seg[a], h.group_seg[b], tiles);
            std::printf("%d %.0f %.0f\n", tiles, s.ragged * tiles, s.off_lines * 1e6);
        } else {
            return 1;
        }
    }
    return 0;
}
