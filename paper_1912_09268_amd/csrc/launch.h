// How a launch is cut up and paced: the rules that turn what a call covers and what the caller has fixed into a grid, a
// form of the kernel and a cap on the workgroups per compute unit.  Pure host code (not part of the C ABI).
#ifndef MGWFBP_LAUNCH_H
#define MGWFBP_LAUNCH_H

#include <algorithm>
#include <cstddef>
#include <cstdint>

#include "mgwfbp.h"
#include "tables.h"

#ifndef MGWFBP_PACK_TILES
#define MGWFBP_PACK_TILES 2       // consecutive full tiles of one tensor that PACK copies in one step
#endif
#define MGWFBP_MAXSEG (2 * MGWFBP_BLOCK)   // segments per tile whose offsets are staged in LDS (two per lane)

namespace {

constexpr int BLOCK = MGWFBP_BLOCK;
constexpr int VEC = MGWFBP_VEC;
constexpr int TVECS = MGWFBP_TILE_VECS;
constexpr int TILE = MGWFBP_TILE_ELEMS;
constexpr int MAXSEG = MGWFBP_MAXSEG;
constexpr int PACK_TILES = MGWFBP_PACK_TILES;

enum Kind { K_PACK = 0, K_REDUCE = 1, K_UPDATE = 2, K_REDUCE_UPDATE = 3, K_PIPELINE = 4, K_DIRECT = 5,
            // what kinds are in kernels of the form THROUGH
            K_REDUCE_UPDATE_THROUGH = 6, K_PIPELINE_THROUGH = 7, K_DIRECT_THROUGH = 8 };

constexpr bool through(int k) { return k >= K_REDUCE_UPDATE_THROUGH; }
constexpr bool reduce_updates(int k) { return k == K_REDUCE_UPDATE || k == K_REDUCE_UPDATE_THROUGH; }
constexpr bool pipelines(int k) { return k == K_PIPELINE || k == K_PIPELINE_THROUGH; }
constexpr bool directs(int k) { return k == K_DIRECT || k == K_DIRECT_THROUGH; }
constexpr bool reads_grads(int k) { return k == K_PACK || pipelines(k) || directs(k); }
constexpr bool reads_merge(int k) { return k == K_REDUCE || reduce_updates(k); }
constexpr bool writes_merge(int k) { return k == K_PACK || pipelines(k); }
constexpr bool sums(int k) { return k == K_REDUCE || reduce_updates(k) || pipelines(k) || directs(k); }
constexpr bool writes_reduced(int k) { return k == K_REDUCE || pipelines(k) || directs(k); }
constexpr bool updates(int k) { return k == K_UPDATE || reduce_updates(k) || pipelines(k) || directs(k); }
constexpr bool needs_owner(int k) { return k != K_REDUCE; }

// Forms of the fast path, beside the number of vectors per lane of a paced step (1 and up).
constexpr int BURST = 0;              // every load of a tile under way at once
constexpr int PAIRS = -1;             // two full tiles of one tensor in one step, single ones in paced steps of one vector
constexpr int THROUGH = -3;           // binary32 pipelines, reduce_updates and direct updates in paced steps of one vector that write through the L2, see goes_through()
constexpr int kind_in(int kind, int form) {
    if (form == THROUGH) return kind == K_REDUCE_UPDATE ? K_REDUCE_UPDATE_THROUGH : kind == K_PIPELINE ? K_PIPELINE_THROUGH : K_DIRECT_THROUGH;
    return kind;
}
constexpr int ON_LINES = -2;          // UPDATE and DIRECT in paced steps of one vector that begin on lines of the weights, see on_lines_pays()
constexpr bool single_steps(int form) { return form == 1 || form == ON_LINES || form == THROUGH; }
constexpr int PAIR = 2;
constexpr int PAIRED = PAIR * TILE;   // elements of a pair
// What needs tiles of one vector per lane, and of one wavefront, is left out of builds with other tiles.
constexpr bool HAVE_PAIRS = TVECS == 1;
constexpr bool HAVE_FEW = TVECS == 1 && BLOCK == 64;
constexpr bool HAVE_PIECES = TVECS == 1 && BLOCK == 64;
// Most segments of a tile that the table form takes piece by piece; the walk over the pieces costs 0.15 us each, the general
// path's prefix sum and search the same for any number.  us with one, up to three and up to eight, 8 workers, tensors in
// groups of eight and more: of 301 elements pipeline 7.2 / 6.4 / 6.4, unpack_update 4.6 / 4.0 / 4.0; of 70 elements pipeline 7.4 /
// 7.3 / 7.0, pack 8.7 / 8.7 / 7.8; of 20 elements (13 pieces, so the general path throughout) 4.5 / 4.5 / 4.5.
#ifndef MGWFBP_PIECES
#define MGWFBP_PIECES 8
#endif
// Kinds whose wavefronts have too little under way with one tile can take joined steps: PACK, a plain copy, always, and
// the pipeline on 16-bit gradients, where a worker's share of a tile is 512 bytes, in kernels of their own: beside the
// joined step, whose sums change hands through LDS, the single-tile kernel would need the joined one's 96 registers instead of 59 (16
// workers; 63 instead of 43 with 8) and as uncapped launches hold 20 instead of 24 wavefronts per compute unit (16
// workers, 6000 tiles: 30.0 us against 23.4, at 16 against 24 wavefronts).
constexpr int joined_tiles_of(int kind, int form) { return form == PAIRS ? PAIR : kind == K_PACK && form != BURST ? PACK_TILES : 1; }

// Dynamic LDS per workgroup that lets at most n workgroups share the 160 KiB of a compute unit.  A workgroup's
// LDS (static + dynamic) is granted in blocks of 1280 bytes (a 128th of the compute unit's; seen in the cap
// sweeps, where 12 and 13, 14 and 15, 16 and 17 behave alike); the total aimed at is the smallest multiple of
// the block above 160 KiB / (n + 1), so n + 1 workgroups never fit, and n do wherever a multiple of the block
// lies in (160 KiB / (n + 1), 160 KiB / n]: 32, 25, 21, 18, 16, 14, 12, 11, 10, 9, 8, ... are the caps that
// exist, and a request in between gets the next lower one.  The request stays 64 bytes short of that total so
// that padding of the static part cannot push it into the next block.  62 KiB keeps clear of the 64 KiB a launch may
// ask for without special arrangements (so n = 1 is served as n = 2).  n <= 0 means no cap, and so does an n beyond
// what the waves of a compute unit allow anyway.
inline size_t lds_for_workgroups_per_cu(int32_t n, size_t static_lds) {
    constexpr int32_t MAX_WGS = 32 * 64 / BLOCK;         // 32 waves per compute unit
    if (n <= 0 || n >= MAX_WGS) return 0;
    if (n < 2) n = 2;
    constexpr size_t CU_LDS = 160u << 10;
    constexpr size_t GRAIN = 1280;
    size_t total = (CU_LDS / static_cast<size_t>(n + 1) / GRAIN + 1) * GRAIN;
    total = std::min<size_t>(total, 62u << 10);
    if (total <= static_lds + 64 + GRAIN) return 0;
    return total - static_lds - 64;
}

// LDS the kernels declare themselves: the table form for its general path (which REDUCE needs only where tiles are not taken
// piece by piece, and less of it), both forms for the sums of joined steps.
constexpr size_t static_lds(int kind, bool few, int form) {
    const size_t joined = form == PAIRS ? sizeof(float) * PAIRED : 0;
    return few || (HAVE_PIECES && !needs_owner(kind)) ? joined : joined + sizeof(int) * static_cast<size_t>((needs_owner(kind) ? 2 * MAXSEG + 1 + BLOCK / 64 : 0) + TILE / VEC + 1);
}

// Default caps, measured on the ResNet-50 shape (25.6 M elements, cold) with every cap that exists, worker counts
// 1, 2, 3, 4, 6, 8, 12, 16, 32 and both gradient widths; GB/s of the cap taken against its neighbours or "none".
//   - What has to be found is the number of bytes a compute unit keeps under way.  A wavefront has N loads in
//     flight, each 1 KiB of a binary32 array or 512 bytes of a 16-bit one: N = 1 in the pipeline, two workers' in
//     the other kinds when P is not known at compile time, all P when it is (2, 4, 8, 16: nothing is stored between
//     them, so the compiler issues them together).
//   - With few workers a wavefront spends more of its life on the way to its first load (header, pointers) than
//     loading, and more of them are needed: REDUCE, binary32, P = 1: 6500 uncapped against 4390 at 14, P = 3: 6278 /
//     5303, P = 4: 6455 at 16 / 6153 uncapped, P = 8: 6562 at 14 / 6258 uncapped.
//   - With many workers there are more arrays to switch between and a smaller window serves them better: pipeline,
//     binary32, P = 4: 6317 at 18 / 6254 at 14, P = 8: 6299 at 14 / 6229 at 16, P = 12: 6260 / 6076, P = 32: 5899 / 5676.
//     That is with the reduced arena; without it there is one array less, and up to 12 workers like 16 better.  ms at 14 / 16, cold
//     and back to back: ResNet-50 shape, P = 6 0.273 / 0.265 and 0.261 / 0.256, P = 8 0.331 / 0.326 and 0.321 / 0.321, P = 12 0.469 / 0.464 and
//     0.461 / 0.465, P = 16 0.604 / 0.611 and 0.600 / 0.610, P = 32 1.159 / 1.194 and 1.170 / 1.199; VGG-16 shape, P = 8 1.777 / 1.767 and 1.778 /
//     1.747; a thousand small layers, P = 12 0.261 / 0.254 and 0.253 / 0.251, P = 16 0.325 / 0.329 and 0.323 / 0.328.
//   - A launch of a few rounds of the chip (the compute units times the cap) should not end in a nearly empty one, see
//     short_launch_cap().
//   - Launches of which more than a quarter of the tiles is ragged are uncapped but with 8 and 16 workers.  The line dates from
//     ragged tiles that took the general path with four workers at a time and needed every wave slot (uncapped over capped with
//     45 % of the tiles ragged, 6 / 12 / 32 workers: pipeline 0.90 / 0.90 / 0.97, direct 0.95 / 0.81 / 0.87).  Piece by piece they hardly do any more:
//     binary32, log-normal sizes around 500 elements in groups of four, 29,000 tiles, 1 / 3 / 6 / 8 / 12 / 16 / 32 workers: pipeline 0.95 / 0.99 / 1.00 /
//     1.04 / 1.02 / 1.02 / 1.02, reduce_update 1.00 / 1.00 / 1.00 / 1.03 / 1.01 / 1.02 / 1.02, direct 1.00 / 1.00 / 0.98 / 1.00 / 0.98 / 1.01 / 1.00; around 1500 elements, 40,000
//     tiles: pipeline 0.99 / 1.01 / 1.01 / 1.04 / 1.04 / 1.03 / 1.05, reduce_update 1.00 / 1.00 / 1.01 / 1.03 / 1.02 / 1.03 / 1.04, direct 0.99-1.01.
//   - 16-bit gradients need every wave slot (direct, P = 8: 6559 uncapped / 5729 at 16), but for launches that would end in a
//     nearly empty round (see even_rounds()), for long REDUCE_UPDATE, which has the registers for 24 to 32 wavefronts (bfloat16, 12 and 150 tensors, us uncapped / at 25: 40,000 tiles P = 4 39.7 / 39.1, 42.1 / 40.3,
//     8 52.6 / 52.5, 54.6 / 54.3, 16 80.1 / 79.9, 82.2 / 82.2; 100,000 tiles P = 4 96.4 / 93.4, 103.6 / 98.3, 8 129.8 / 126.6, 136.0 / 131.9, 16
//     193.3 / 191.5, 201.4 / 199.4; P = 1 level; 12,000 tiles level, 7000 tiles P = 4 8.9 / 9.7, 8 11.4 / 12.6), for REDUCE with all of
//     8 or 16 workers' loads in flight (P = 16: 6381 at 16 / 6220 uncapped; P = 12, two at a time: 6512 / 5265) and
//     for the pipeline's joined steps, which have 1 KiB under way like binary32 (P = 8: 6164 at 14 / 5886 uncapped).
//     The longest of those like a smaller window where they write the reduced arena as well.  us at 12 / 14, P = 8, with it: 46 M
//     elements 390.4 / 389.1, 67 M 553.1 / 561.0, 102 M 859 / 871, 333 M 2831 / 2894, and with a cold memory-side cache 67 M 564 / 567, 102 M
//     882 / 896, 333 M 2881 / 2940; P = 4, 67 M 378.7 / 383.8; P = 16 927.8 / 932.9.  Without it the two are level: 67 M 504.9 / 506.1, 102 M 787 /
//     789, 333 M 2568 / 2589, cold 519.2 / 515.5, 800 / 800, 2630 / 2634.
constexpr int32_t SHORT_LAUNCH_TILES = 16384;
constexpr int32_t LONG_LAUNCH_TILES = 262144;       // 67 M elements

// Longest launch, in tiles, that takes the burst form.  Up to here the time is the latency of a tile, beyond it the
// loads of all tiles at once are more than the memory system likes.  us burst / paced (the pipeline's rolling steps among
// these, see rolls()).
//   binary32, one tensor          1400         1800         2300 tiles
//     pipeline        P = 4    4.9 / 5.2    5.2 / 5.7    7.1 / 7.0
//                         6    5.6 / 6.5    6.7 / 7.2    9.1 / 9.1
//                         8    6.9 / 7.1    8.1 / 8.0   11.6 / 10.9
//                        12    9.1 / 9.3   10.9 / 10.6  15.9 / 14.4
//                        16   11.0 / 10.8  13.5 / 12.5  20.4 / 17.9
//   binary32, 150 equal tensors   1350         1650         1950 tiles
//     reduce          P = 4    2.3 / 2.2    2.4 / 2.3    2.6 / 2.6
//                         6    2.9 / 3.3    3.0 / 3.4    3.2 / 3.4
//                         8    4.0 / 4.0    4.0 / 4.1    4.3 / 4.1
//                        12    4.6 / 5.4    5.0 / 5.6    5.5 / 5.8
//                        16    6.3 / 6.5    6.9 / 6.6    8.4 / 6.9
//                        32   10.7 / 11.8  11.4 / 12.2  12.5 / 12.5
//     reduce_update   P = 4    3.2 / 4.0    3.6 / 4.3    3.9 / 4.4
//                         8    4.6 / 5.4    5.0 / 5.6    5.7 / 5.8
//                        12    5.6 / 7.0    6.2 / 7.3    7.1 / 7.5
//                        16    7.4 / 8.0    8.6 / 8.3    9.7 / 8.4
//                        32   11.7 / 13.2  12.7 / 13.7  13.6 / 14.2
//   binary32, one tensor          1024         1792         2560 tiles
//     direct          P = 4    3.2 / 4.3    4.0 / 4.9    5.2 / 5.5
//                         8    3.9 / 5.4    5.2 / 6.2    6.6 / 6.9
//                        12    4.9 / 6.8    6.5 / 7.9    8.2 / 8.7
//                        16    5.3 / 7.5    7.6 / 8.7   10.1 / 9.9
//                        32    8.2 / 12.9  11.6 / 14.5  16.3 / 16.1
//   one tensor                    3072         4096 tiles
//     binary32 pipeline P = 1, 2, 3        5.3 / 6.0, 6.0 / 6.3, 7.5 / 6.6      6.6 / 7.0, 8.2 / 8.0, 10.0 / 9.5
//     binary32 update                      4.5 / 4.6                            5.6 / 5.4
//     bfloat16 pipeline P = 2, 4, 8, 12    5.1 / 5.5, 6.5 / 6.6, 8.9 / 8.7, 11.3 / 10.8    6.9 / 6.9, 9.1 / 9.2, 13.2 / 12.8, 16.9 / 16.4
//     bfloat16 reduce_update P = 3, 8, 12  4.6 / 5.8, 6.0 / 6.6, 6.9 / 8.5      5.8 / 6.6, 8.2 / 7.5, 9.7 / 9.7
//     bfloat16 direct P = 3, 8, 12         4.8 / 5.7, 6.1 / 6.9, 7.0 / 8.5      5.8 / 6.4, 7.5 / 7.8, 9.9 / 9.4
// Where reduce of 8 and 16 workers is level here, other runs have the paced form 3 % ahead (8 workers, 1600 tiles 4.5 / 4.3).
// PACK has one form (every load of a step under way, see joined_tiles); for it this is where the cap begins.
inline int32_t default_burst_tiles(int kind, int32_t dtype, int32_t P) {
    if (kind == K_PACK) return 1024;
    if (dtype != MGWFBP_F32 || P < 4 || kind == K_UPDATE) return 3072;
    if (kind == K_DIRECT) return P == 16 ? 1792 : 2560;
    if (kind == K_REDUCE) return P == 8 || P == 16 ? 1280 : 1792;
    return P != 16 ? 1792 : kind == K_REDUCE_UPDATE ? 1536 : 1280;
}

// Whether a workgroup of the pipeline takes two tiles in one step (see joined_tiles).  GB/s at 16-bit gradients,
// ResNet-50 shape, joined at its best cap against single tiles uncapped: P = 1: 6250 / 6327, 2: 6221 / 6231,
// 3: 6194 / 6127, 4: 6175 / 6038, 8: 6164 / 5881, 16: 6080 / 5737, 32: 5675 / 5554; with one or two workers the
// binary32 arrays are most of the traffic.  A short launch needs its tiles spread over the chip.
// Nor does a model of many ragged tiles, whose turns come one after the other in a pair: with 0.9 / 2 / 3 / 11 / 45 % of
// its tiles ragged, bf16, P = 8: 5706 / 5583 / 5789 / 5408 / 4364 joined, 5528 / 5446 / 5891 / 5532 / 4640 not.
// In launches of up to twice SHORT_LAUNCH_TILES a single ragged tile counts where the worker count is not a compiled one.  That
// dates from ragged tiles that took four workers at a time on the general path (bfloat16, one tensor that ends in a ragged second
// half of a pair, pairs over single tiles, 16,500 tiles 6 / 12 / 32 workers 1.09 / 1.13 / 1.17).  Piece by piece the ragged half costs little: 16,500
// tiles 4 / 6 / 8 / 12 / 16 / 32 workers 1.00 / 0.98 / 1.00 / 0.97 / 1.04 / 0.97, 24,000 0.96 / 0.93 / 0.95 / 0.94 / 0.96 / 0.96, 31,000 0.97 / 0.94 / 0.93 / 0.93 / 0.94 / 0.97;
// without it 1.00 / 0.96 / 0.99 / 0.95 / 1.03 / 0.96, 0.92-0.98, 0.91-0.97.
inline bool joined_pipeline(int32_t dtype, int32_t P, int32_t tiles, double ragged) {
    const bool compiled = P == 4 || P == 8 || P == 16;
    return dtype != MGWFBP_F32 && P >= 3 && tiles >= (compiled || ragged == 0 ? 1 : 2) * SHORT_LAUNCH_TILES && ragged < 0.025;
}

// Tiles per workgroup of a PACK, which copies two of them per step: 4 KiB of a worker's binary32 gradients at 14
// workgroups per compute unit; 2 KiB uncapped where ragged tiles, which are copied one by one, are no rarity (P = 3,
// 0.02 / 0.9 / 2 / 11 / 45 % ragged: 6399 / 6148 / 5829 / 4922 / 2499 with 4 KiB, 6397 / 6188 / 5938 / 5792 / 3745 with 2 KiB);
// 2 KiB of 16-bit gradients (P = 3, same models: 6164 / 5758 / 5110 / 4207 / 2085, with 4 KiB 6022 / 5398 / 4678 / 3684 / 1967).
// Up to 256 copies of tiles per compute unit a launch is over sooner with more workgroups (f32, us with 1 / 2 / 4
// tiles each: P = 8, 1024 tiles 5.4 / 5.0 / 5.5, 4096 tiles 16.0 / 12.5 / 13.1, 16384 tiles 64.9 / 42.9 / 42.2; P = 1, 1024
// tiles 2.9 / 2.9 / 3.4).  Up to 8 per compute unit two are no faster than one, and slower where the ends of what is
// packed are ragged (a thousand tensors around 4096 elements as views, packed one by one: 6222 us with 2, 5877 with 1).
// With 16-bit gradients of many workers, next to no ragged tiles and a million copies of tiles 4 KiB at 21 workgroups per
// compute unit are ahead (ResNet-50 shape, 0.017 % ragged, us: P = 32: 493 against 510 with 2 KiB uncapped, P = 16: 248 / 257, P = 8:
// 127 / 128; one tensor of 100,000 tiles P = 24: 373 / 382, P = 12: 186 / 190, P = 8: 125 / 125).  Not in shorter launches (30,000
// tiles P = 8 / 16 / 24: 40.4 / 38.9, 75.9 / 74.0, 112.8 / 112.7; 10,000 tiles 16.0 / 14.8, 28.6 / 27.0, 40.4 / 38.9), nor reliably with more
// ragged tiles (100,000 tiles, 0.05 / 0.1 / 0.2 / 1 %: P = 16 270.7 / 269.0, 273.3 / 266.7, 264.9 / 267.6, 280.2 / 273.9).
constexpr double SOME_RAGGED = 0.005, HARDLY_RAGGED = 0.0004;
constexpr int64_t SINGLE_COPIES = 2048, FEW_COPIES = 65536, MANY_COPIES = 1 << 20;
inline bool many_halves(int32_t dtype, int32_t P, int64_t copies, double ragged) {
    return dtype != MGWFBP_F32 && P >= 12 && copies > MANY_COPIES && ragged < HARDLY_RAGGED;
}
inline int32_t pack_tiles_per_workgroup(int32_t dtype, int32_t P, int64_t copies, double ragged) {
    if (copies <= SINGLE_COPIES) return 1;
    if (many_halves(dtype, P, copies, ragged)) return 8;
    return copies <= FEW_COPIES || (dtype == MGWFBP_F32 && ragged > SOME_RAGGED) ? 2 : 4;
}

inline int32_t default_workgroups_per_cu(int kind, int32_t dtype, int32_t P, int32_t tiles, double ragged, bool reduced, int form) {
    const bool wide = dtype == MGWFBP_F32;
    if (ragged > 0.25 && kind != K_REDUCE && (kind == K_PACK || (P != 8 && P != 16))) return -1;
    switch (kind) {
        case K_REDUCE: return wide ? (P < 4 ? -1 : P < 8 ? 16 : 14) : (P == 8 || P == 16 ? 16 : -1);
        case K_UPDATE: return -1;                        // 20 bytes per element, nothing per worker
        case K_PACK:
            if (many_halves(dtype, P, static_cast<int64_t>(tiles) * P, ragged)) return 21;
            if (!wide || ragged > SOME_RAGGED) return -1;
            return tiles < SHORT_LAUNCH_TILES ? 18 : 14;
        case K_REDUCE_UPDATE: return wide ? (P < 4 ? 25 : P < 8 ? 16 : 14) : P >= 4 && P <= 16 && tiles >= 2 * SHORT_LAUNCH_TILES ? 25 : -1;
        case K_DIRECT: return wide ? (P < 4 ? 25 : P <= 8 ? 16 : 14) : -1;
        default:                                         // pipeline
            if (wide) return P < 6 ? 18 : !reduced && P <= 12 ? 16 : 14;
            if (form != PAIRS || tiles < SHORT_LAUNCH_TILES) return -1;
            return tiles < LONG_LAUNCH_TILES || !reduced ? 14 : 12;
    }
}

// The cap of a launch of a few rounds, binary32 or in pairs of tiles, next to the `cap` of long ones: all workgroups at
// once where 25 per compute unit hold them (16 workers, but for REDUCE: 20 in the few-segments form, by its registers, 16 in the
// table form and in pairs, which date from kernels that held 16; binary32 ones hold 20 now: us as launched / at once, 150 tensors of
// 4200 / 4650 / 5100 tiles, pipeline 33.9 / 28.0, 35.9 / 31.2, 36.7 / 33.5, reduce_update 19.1 / 15.1, 19.8 / 17.4, 20.5 / 19.3, direct 18.6 / 14.9, 18.7 / 16.1,
// 19.5 / 17.2, but 5400 37.5 / 41.2, 21.2 / 24.1, 19.5 / 21.6), else the neighbour whose rounds come out fullest.  Pipeline, 8 workers, one tensor of 5000 tiles (19.5 per compute unit): 21.4 / 22.1 / 22.5 us in two
// rounds at 14 / 16 / 18, 19.1 in one.  Per cent above the best of 14 / 16 / 18 / 21, mean of reduce, direct and pipeline with
// 8, 12, 16 and 32 workers: 7100 tiles 0.2 / 0.7 / 2.9 / 5.0, 7200 12.0 / 0.3 / 1.9 / 3.4, 8250 6.0 / 9.4 / 0.0 / 1.7, 9250 0.3 / 4.2 / 7.8 /
// 1.8, 11000 7.5 / 0.0 / 2.3 / 6.6, 13000 1.4 / 5.3 / 0.3 / 2.2, 13900 0.5 / 2.8 / 5.7 / 1.9, 18000 2.3 / 1.5 / 0.4 / 3.0, 24000 0.9 / 0.2 /
// 3.0 / 2.4.  The longer a tile takes and the more rounds there are, the more these blur (direct, 8 workers, 65,000 tiles:
// 123.7 us at the cap of long launches, 127.8 at the fuller neighbour; pipeline, 32 workers, 18,000 tiles 219.8 / 227.8,
// 16,000 184.5 / 184.1; 12 workers, 40,000 tiles 192.0 / 189.0).  Pairs, bfloat16, 16,000 tiles at 14 / 16 / 18: 8 workers 38.7 / 36.3 /
// 37.1 us, 32 workers 111.1 / 100.9 / 103.2; 40,000 tiles 86.2 / 87.0 / 87.7, 253.3 / 254.1 / 262.8.  A cap that suits few
// workers (25, none) holds at any length.
inline bool few_rounds(int32_t tiles, int32_t P) { return tiles < 49152 && static_cast<int64_t>(tiles) * P < 500000; }
inline int32_t short_launch_cap(int32_t cap, int kind, int32_t P, bool few, int32_t per_cu) {
    if (cap <= 0 || cap >= 25) return cap;
    const int32_t most = P != 16 || kind == K_REDUCE ? 25 : few ? 20 : 16;
    if (per_cu <= most) return 25;
    auto slots = [&](int32_t n) { return (per_cu + n - 1) / n * n; };      // of all rounds, per compute unit
    auto fuller = [&](int32_t a, int32_t b) { return slots(a) <= slots(b) ? a : b; };
    if (cap >= (kind == K_PIPELINE ? 18 : 16)) return fuller(18, 21);
    return most < 18 ? fuller(14, 16) : fuller(fuller(14, 16), 18);
}

// Units per die and turn (log2), where tiles start inside lines (see unit_of): the kinds that write w and v gain,
// the pipeline, which writes whole lines of P arenas as well, less; PACK and REDUCE write whole lines only.  `off_lines` is the
// share of the elements of tensors off their lines, as far as sizes and places in the arena show it: a tensor of odd size
// that begins its group lies off its lines as a view of a flat buffer (100,000 tiles: pipeline 0.91-0.99 of the time with runs,
// direct 0.83-0.92), but on them in an allocation of its own (pipeline 0.99-1.02, direct and reduce_update 0.95-1.05).  Time with
// runs over that without by share, binary32, 60,000 tiles, 0.1 / 0.3 / 0.45 / 0.7 / 1: pipeline 3 workers 1.00 / 0.99 / 0.98 / 0.96 / 0.94, 8
// workers 1.00 / 0.99 / 0.99 / 0.97 / 0.97; update 0.99 / 0.98 / 0.97 / 0.94 / 0.94; direct 3 workers 1.00 / 0.98 / 0.96 / 0.91 / 0.90, 8 workers
// 1.02 / 1.00 / 0.98 / 0.94 / 0.90, 16 workers 1.03 / 1.01 / 0.99 / 0.95 / 0.93; reduce_update 3 workers 1.01 / 1.00 / 0.98 / 0.94 / 0.93, 8
// workers 1.02 / 1.02 / 1.01 / 0.99 / 0.97, 16 workers 1.04 / 1.03 / 1.04 / 1.01 / 1.01, 32 workers 1.05 at 1; bfloat16, 8 workers, at most 1.00
// throughout.
inline int8_t run_log2_of(int kind, int32_t dtype, int32_t P, double off_lines) {
    if (kind == K_PACK || kind == K_REDUCE) return 0;
    const bool wide = dtype == MGWFBP_F32;
    const int32_t bytes = P * (wide ? 4 : 2);             // of gradients per element
    if (kind == K_REDUCE_UPDATE && bytes > 32) return 0;
    const bool late = wide && bytes >= 32 && (kind == K_REDUCE_UPDATE || kind == K_DIRECT);
    if (off_lines <= (late ? 0.5 : 0.25)) return 0;
    return kind == K_PIPELINE ? 2 : 3;
}

// Shares of tiles that begin on lines of the weights.  A tile is 256 elements of the arena, and a tensor of odd size, or after one, lies
// somewhere else in its lines of 128 bytes: a wavefront then touches nine lines of w, v and every worker's gradients for eight (five for
// four of 16-bit gradients), neighbours fetch the line they share twice and each write a part of it.  UPDATE and DIRECT, which touch the arenas
// not at all or only to read the reduced one, need not cut a tensor where its tiles are: inside a tensor a tile's share begins at the last line
// before its first element, and ends where the next tile's begins.
//   line_shift: elements from there to the tile's first element; address of the tensor's weights, its start as seen from the tile
//   starts_early: what the share really begins earlier by, no earlier than the tensor (first_start: 0 where it begins with the tile)
constexpr int line_shift(uint64_t weights, int64_t first_start, int line) {
    return static_cast<int>(weights / sizeof(float) - static_cast<uint64_t>(first_start)) & (line - 1);
}
constexpr int starts_early(int64_t first_start, int shift) { return -first_start < shift ? static_cast<int>(-first_start) : shift; }
constexpr int line_elems(int kind, size_t grad_bytes) { return 128 / static_cast<int>(kind == K_DIRECT ? grad_bytes : sizeof(float)); }

// Where that pays: time over tiles cut in the arena with runs of tiles per die (see above).  300 tensors of log-normal odd sizes, views of flat
// buffers / allocations of their own in groups of five / a group each (where every tensor begins on a line and nothing is gained) / views of
// sizes that are multiples of 64:
//   binary32   update  8000 tiles 0.98 / 0.97 / 1.02 / 1.00    20,000 0.98 / 0.97 / 1.02 / 1.00    100,000 0.94 / 0.94 / 1.00 / 1.01
//              direct, 1 worker   8000 0.95 / 0.94 / 1.01 / 1.01    20,000 0.98 / 0.95 / 1.01 / 1.01    100,000 0.96 / 0.97 / 1.00 / 1.01
//                      3 workers  8000 0.96 / 0.97 / 1.04 / 1.01    20,000 0.97 / 0.97 / 1.01 / 1.00    100,000 0.96 / 0.96 / 0.99 / 1.00
//                      8 workers  8000 0.99 / 1.02 / 1.04 / 1.00    20,000 0.97 / 0.99 / 1.01 / 1.00    100,000 0.96 / 0.97 / 0.98 / 1.00
//   bfloat16   direct, 3 workers  8000 0.95 / 0.95 / 1.03 / 1.00    20,000 0.95 / 0.95 / 1.00 / 1.00    100,000 0.93 / 0.95 / 1.00 / 1.00
//                      8 workers  8000 0.94 / 0.97 / 1.02 / 1.00    20,000 0.91 / 0.93 / 1.01 / 1.00    100,000 0.92 / 0.93 / 1.01 / 1.00
//                      16 workers 8000 0.87 / 0.93 / 1.03 / 1.00    20,000 0.84 / 0.90 / 1.01 / 1.00    100,000 0.88 / 0.91 / 1.00 / 1.00
// (those without runs; see runs_on_lines()).  With 12,000 tensors of 100,000 tiles, update 0.97 / 0.98 / 1.01 / 1.01, direct 8 workers 0.97 / 0.98 / 1.02 / 1.02 and
// bfloat16 0.93 / 0.94 / 1.02 / 1.01; the tiles a tensor begins or ends in take a step more.  The lines lie where a group each in allocations of their own, which the
// host takes for views, no longer pays: at 24,600 tiles update 1.00, direct binary32 1 / 3 / 8 / 16 workers 1.01 / 1.00 / 1.00 / 1.00, bfloat16 at 16,400 1.00-1.01 (4 workers
// between 18,500 and 25,500 tiles 0.98-1.05, the others 1.00-1.01).
// Over the few tensors of the few-segments form, against that form, one large odd one behind a small one / five as views / five in allocations of their own:
//   16,400 tiles  direct, bfloat16 1 / 4 / 8 / 16 workers 0.97 / 0.98 / 0.98, 0.91 / 0.97 / 0.96, 0.86 / 0.97 / 0.92, 0.79 / 0.95 / 0.86
//   20,000        the same 0.98 / 0.98 / 0.98, 0.95 / 0.99 / 0.98, 0.91 / 0.99 / 0.96, 0.82 / 0.94 / 0.89
//   24,600        the same 0.96 / 0.97 / 0.98, 0.92 / 0.94 / 0.94, 0.90 / 0.91 / 0.93, 0.82 / 0.88 / 0.89; binary32 update 0.96 / 0.99 / 0.98, direct 1 / 8 / 16 workers 0.97 /
//                 0.97 / 0.98, 0.95 / 0.95 / 0.95, 0.92 / 0.96 / 0.94
//   40,000        the same 0.94 / 0.95 / 0.97, 0.89 / 0.92 / 0.93, 0.86 / 0.90 / 0.90, 0.79 / 0.87 / 0.85; 0.95 / 0.97 / 0.97, 0.95 / 0.95 / 0.96, 0.94 / 0.93 / 0.94, 0.95 / 0.94 / 0.93
// Eight odd tensors, a group each, in allocations of their own pay up to 4 % with bfloat16 of up to 8 workers to 24,600 tiles (20,000: 1 / 4 / 8 workers 1.03-1.04 / 1.02 /
// 1.01-1.03) and gain 0-5 % from 30,000 on; as views of one buffer, for which they are taken, they gain from 16,400 on (20,000: 0.98 / 0.96 / 0.94, 16 workers 0.89).
// The pipeline would have its arenas off the lines instead (0.84-0.97 of the rate), reduce_update gains with one or two 16-bit workers only.
inline bool on_lines_pays(int kind, int32_t dtype, bool reduced, int32_t tiles, int32_t segments, double off_lines) {
    if (kind != K_UPDATE && (kind != K_DIRECT || reduced)) return false;
    const int32_t least = kind == K_DIRECT && dtype != MGWFBP_F32 ? SHORT_LAUNCH_TILES : SHORT_LAUNCH_TILES / 2 * 3;
    return off_lines > 0.25 && tiles >= least && tiles / 16 >= segments;
}

// Which of the launches that could take the few-segments form do.  It reaches a ragged tile's data several memory trips
// sooner (a launch of up to 1000 tiles over five tensors takes 0.76-0.9 of the table form's time, over one tensor that ends in a
// ragged tile 0.9-1.0), but full tiles cost it a little more, and that adds up where every wavefront counts.  Time over that
// of the table form, launches over one tensor unless said otherwise:
//   - REDUCE has no ragged tiles but at the groups' ends: 0.94-1.04 up to 2000 tiles; 1 worker at 3500 / 14000 / 60000 tiles
//     binary32 1.08 / 1.10 / 1.09, bfloat16 1.05 / 1.17 / 1.26, 3 workers bfloat16 1.09 / 1.14 / 1.16.
//   - 16-bit PACK, 2 workers: copies of tiles up to 4096 1.05-1.10 (ragged end: 0.95), 7000 / 18000 / 48000 1.11 / 1.12 / 1.08
//     (1.00 / 1.03 / 1.06), beyond 65536 0.97-1.00.
//   - The other kinds on 16-bit gradients, which run uncapped.  Most few-segments kernels have registers for 32 wavefronts per
//     compute unit, and most table kernels for 24 or 28, so that 25 to 32 tiles per compute unit run at once, and 49 to 56 in
//     two rounds, in this form only: 2 / 4 / 8 / 16 / 32 workers, 6300 tiles direct 0.96 / 0.96 / 0.80 / 0.81 / 0.74, reduce_update 0.97 / 0.97 / 0.97 /
//     0.78 / 0.73, pipeline 0.97 / 0.99 / 0.98 / 0.98 / 0.96, 7900 tiles direct 0.90 / 0.87 / 0.88 / 0.91 / 0.84, reduce_update 0.98 / 0.97 / 0.85 / 1.02 / 0.82;
//     12,600 tiles direct 0.98 / 0.98 / 0.90 / 0.93 / 0.90, reduce_update 0.99 / 0.98 / 0.98 / 0.91 / 0.91.  Elsewhere it goes either way: 4700 tiles direct
//     0.96 / 0.95 / 0.96 / 0.99 / 0.98, 8300 0.96 / 0.97 / 1.03 / 1.07 / 1.06, 17,000 1.01 / 1.00 / 1.05 / 1.08 / 1.10, reduce_update 0.94 / 0.96 / 0.95 / 0.97 / 0.98, 0.99 /
//     0.98 / 0.99 / 1.03 / 1.06, 1.00 / 0.99 / 1.03 / 1.03 / 1.08 (without the cap of even_rounds()).  Over five tensors 0.9-1.03.
//   - binary32: 0.95-1.04 over one tensor, 0.9-1.02 over five.
constexpr int FEW = 8;                // segments that fit into a launch's arguments
inline bool few_form_pays(int kind, int32_t dtype, int32_t P, int32_t tiles, int32_t segments, int32_t per_cu) {
    if (kind == K_REDUCE) return tiles <= 2048;
    if (dtype == MGWFBP_F32 || segments > 1) return true;
    const int64_t copies = static_cast<int64_t>(tiles) * P;
    if (kind == K_PACK) return copies <= 4096 || copies > FEW_COPIES;
    return tiles <= 3072 || (per_cu > 24 && per_cu <= 32) || (per_cu > 48 && per_cu <= 56);
}

// Which of the launches that begin on lines have runs of tiles per die all the same.  No line is shared any more; that runs still pay in some
// of them is what the times say.  Time with runs over without, 300 tensors as views / in allocations of their own in groups of five / a group
// each / eight tensors a group each, at 30,000, 50,000 (without the groups of five), 70,000 and 140,000 tiles:
//   update                     0.986 / 0.978 / 1.002 / 1.007    0.977 / 0.996 / 1.006    0.970 / 0.978 / 0.987 / 1.002    0.976 / 0.984 / 1.014 / 1.009
//   direct  binary32, 1        0.996 / 0.993 / 1.003 / 1.014    0.983 / 0.990 / 1.015    0.959 / 0.960 / 0.955 / 0.998    0.975 / 0.976 / 0.975 / 1.005
//           binary32, 3        1.000 / 0.996 / 1.002 / 1.020    1.007 / 1.012 / 1.021    1.001 / 1.005 / 0.999 / 1.012    1.019 / 1.030 / 1.030 / 1.023
//           binary32, 8        1.004 / 1.000 / 1.013 / 1.030             -               1.020 / 1.031 / 1.022 / 1.034    1.016 / 1.027 / 1.036 / 1.037
//           bfloat16, 1        0.986 / 0.993 / 1.006 / 1.026    0.979 / 0.993 / 1.006    0.961 / 0.961 / 0.955 / 0.983    0.968 / 0.967 / 0.971 / 0.987
//           bfloat16, 3        0.994 / 1.002 / 1.004 / 1.012    0.981 / 0.991 / 1.011    0.962 / 0.967 / 0.962 / 0.983    0.975 / 0.974 / 0.976 / 0.996
//           bfloat16, 8        0.993 / 0.997 / 1.002 / 1.015    0.990 / 0.993 / 1.006    0.979 / 0.981 / 0.981 / 0.992    0.990 / 0.988 / 0.996 / 0.998
//           bfloat16, 16       0.996 / 0.997 / 1.003 / 1.014    0.989 / 0.990 / 1.024    0.988 / 0.986 / 0.992 / 1.000    0.989 / 0.991 / 0.991 / 1.005
//           bfloat16, 32       0.994 / 0.998 / 1.002 / 1.041             -               0.981 / 0.985 / 0.993 / 0.995    0.994 / 0.995 / 0.988 / 1.008
// Few tensors gain less: eight a group each and five as views at 52,000 tiles 1.00-1.02 throughout, at 70,000 and 100,000 update 1.002 / 0.982, 1.012 / 0.980, bfloat16
// 8 workers 0.997 / 0.999, 1.009 / 0.997, 16 workers 1.002 / 1.018, 1.016 / 1.018, binary32 of one worker 0.99-1.00, at 200,000 1.008 /
// 1.014.  Updates of 200,000 tiles are 0.984 / 0.985 / 1.029 / 1.022, other direct steps of one worker level again.  Time over the
// tiles cut in the arena with their runs, a group each in allocations of their own, which are on lines in truth, 60,000 to 140,000 tiles: direct binary32 of one
// worker and bfloat16 of 1 to 6 1.02-1.055 without runs here, 1.00 with them.  Where some of the weights and momenta are kept cacheable (64 MiB of them, 100,000
// tiles) runs bring nothing (1.00-1.03, five tensors bfloat16 4 workers 1.05).
inline bool runs_on_lines(int kind, int32_t dtype, int32_t P, int32_t tiles, int32_t segments) {
    const bool few = segments <= FEW;
    if (tiles < (few ? 4 : 3) * SHORT_LAUNCH_TILES) return false;
    if (kind == K_UPDATE) return !few && tiles <= LONG_LAUNCH_TILES / 2;
    return dtype == MGWFBP_F32 ? P == 1 && !few : P <= (few ? 7 : 16);
}

// Kernels with rolling steps beside the single ones (see rolling_tile).
constexpr bool may_roll(int kind, int form) { return TVECS == 1 && kind == K_PIPELINE && form == 1; }
constexpr bool compiled(int32_t P) { return P == 2 || P == 4 || P == 8 || P == 16; }
// Wavefronts per compute unit that the pipeline's single-tile kernels on 16-bit gradients have registers for.
inline int32_t pipeline_wavefronts(int32_t P, bool few) {
    if (P == 16) return 24;
    if (few) return P == 8 ? 28 : 32;
    return P == 2 ? 28 : compiled(P) ? 24 : 32;
}
// Launches of the pipeline in single tiles whose wavefronts, with one load each, have too little under way between them: binary32
// up to 12 per compute unit, 16-bit gradients, whose loads are half as long, up to 16, and where a second round of them is
// nearly empty.  Time of rolling steps over that of single ones, one tensor (few-segments form) / 150 equal tensors / 12 as views /
// 300 of log-normal sizes as views (table form); thousands of tensors of some hundred elements are at 11 per compute unit 0.96 with 8
// workers and 0.93 with 16:
//   binary32     8 per CU  P = 4 0.84 / 0.84 / 0.84 / 0.94, 8 0.85 / 0.82 / 0.84 / 0.87, 12 0.91 / 0.90 / 0.90 / 0.91, 16 0.84 / 0.80 / 0.84 / 0.89
//               10         P = 4 0.92 / 0.91 / 0.95 / 0.99, 8 0.98 / 0.90 / 0.98 / 1.00, 12 0.95 / 0.93 / 0.96 / 0.96, 16 1.00 / 0.94 / 1.00 / 1.01
//               12         P = 4 0.99 / 0.93 / 0.98 / 1.05, 8 1.00 / 0.96 / 1.00 / 1.02, 12 0.97 / 0.95 / 0.97 / 0.98, 16 1.00 / 0.99 / 1.03 / 1.00
//               13         P = 4 1.04 / 0.99 / 1.04 / 1.04, 8 1.05 / 1.01 / 1.05 / 1.04, 12 0.97 / 0.96 / 0.98 / 0.97, 16 1.05 / 1.05 / 1.08 / 1.04
//   bfloat16    16         P = 2 0.93 / 0.93 / 0.95 / 1.04, 4 0.93 / 0.92 / 0.94 / 1.01, 8 0.91 / 0.89 / 0.93 / 1.01, 16 0.88 / 0.87 / 0.92 / 0.97
//               26         P = 2 0.99 / 0.99 / 1.00 / 1.02, 4 1.05 / 0.89 / 0.91 / 0.95, 8 1.06 / 0.87 / 0.91 / 0.93, 16 0.90 / 0.85 / 0.90 / 0.93
//               30         P = 2 0.98 / 0.94 / 0.96 / 0.99, 4 1.02 / 0.92 / 0.96 / 0.97, 8 0.94 / 0.89 / 0.94 / 0.96, 16 0.91 / 0.88 / 0.95 / 0.97
//               34         P = 2 0.98 / 0.97 / 0.96 / 1.01, 4 0.97 / 0.97 / 1.00 / 1.01, 8 0.96 / 0.96 / 0.99 / 1.00, 16 0.96 / 0.96 / 0.99 / 1.00
//               36         P = 2 0.99 / 0.98 / 0.99 / 1.03, 4 0.98 / 0.98 / 1.00 / 1.04, 8 1.01 / 0.96 / 1.00 / 1.01, 16 1.01 / 0.97 / 1.01 / 1.01
// (At 34 and 36 one tensor takes the table form, too; a little below 36, at 9000 tiles on 256 compute units, 8 workers gain 4 %, 16
// 3 %.)  Where the worker count is not compiled single steps hold 32 wavefronts: 12 workers at 26 / 30 0.99 / 1.01, 32 over 12
// tensors at 30 1.11.  At 33 to 36, with the cap of even_rounds() in both: 6 / 12 / 32 workers over five tensors 0.95 / 0.96 / 0.95, 150 0.95 /
// 0.95 / 0.95, 12 as views 0.96 / 0.96 / 0.96, log-normal 0.96 / 0.95 / 0.96.
inline bool rolls(int32_t dtype, int32_t P, bool few, int32_t per_cu) {
    if (dtype == MGWFBP_F32) return per_cu <= (P == 8 || P == 16 ? 11 : few || compiled(P) ? 12 : 10);
    return per_cu <= 16 || (per_cu > pipeline_wavefronts(P, few) && per_cu <= 36);
}

// 16-bit gradients in single tiles run uncapped, but a launch that takes as many rounds of the chip with 24 wavefronts per
// compute unit as with the 32 (or 28) there are registers for does not fill the last of these.  Time at the cap of 25 (24 of such a
// kernel) over uncapped, bfloat16, tiles per compute unit in brackets: pipeline over 150 tensors, 6 / 12 / 32 workers (34) 0.99 / 0.96 / 0.94, (37)
// 0.95 / 0.92 / 0.91, (39) 0.96 / 0.93 / 0.89, (45) 0.99 / 0.96 / 0.92, but (49) 1.01 / 0.99 / 0.97, (53) 1.08 / 1.08 / 1.08; over five, 12 workers (37) 0.93, (45) 0.95, (53)
// 1.08; reduce_update over 150, 4 workers (34) 0.94, (37) 0.95, (45) 0.99, (53) 1.05, (67) 0.97, (71) 0.98, (80) 1.03; 16 workers, 28 wavefronts, (29)
// 0.98, (64) 0.97, (74) 0.98, (80) 1.05; direct over five, 8 / 16 workers (34) 0.94 / 0.93, (37) 0.97 / 0.96, (45) 0.98 / 0.97, (53) 1.08 / 1.11.  Kernels with registers
// for 24 do not mind; the pipeline's of 2 to 16 workers, in part such, would lose 1-5 % at 34.
inline bool even_rounds(int kind, int32_t dtype, int32_t P, bool few, int form, int32_t per_cu) {
    if (dtype == MGWFBP_F32 || form != 1) return false;
    if (kind != K_REDUCE_UPDATE && kind != K_DIRECT && !(kind == K_PIPELINE && !compiled(P))) return false;
    const int32_t held = kind == K_REDUCE_UPDATE && !few && (P == 16 || (P == 8 && dtype == MGWFBP_F16)) ? 28 : 32;
    return per_cu > held && (per_cu + held - 1) / held == (per_cu + 23) / 24;
}

// Results are streamed by every kind, also those that the next step reads.  Ordinary stores would leave them in the 256 MB memory-side cache, but
// that pays only where nothing lies between the steps, and then reduce_update or the pipeline does them in one pass; a caller of single steps has
// the exchange in between, and PACK and REDUCE themselves take longer.  Time with ordinary stores over streamed, repeated
// over three sets of buffers | from an emptied cache:
//   REDUCE, 150 even tensors, reduced arena of 120 / 200 / 300 / 500 MiB
//     binary32 1 worker    by itself 1.00 / 1.02 / 1.04 / 1.03 | 0.96 / 0.95 / 0.95 / 0.96, unpack_update right after it 0.95 / 0.94 / 0.95 / 0.99 | 0.98 / 0.97 / 0.98 /
//                          1.00, a copy of the arena in between 1.04 / 1.05 / 1.01 / 1.02 | 0.92 / 1.02 / 1.02 / 1.01
//     binary32 4 workers   1.04 / 1.05 / 1.04 / 1.03 | 1.00 / 1.00 / 1.00 / 0.99, 0.96 / 0.96 / 0.98 / 1.00 | 1.00 / 0.99 / 1.00 / 1.01, 1.04 / 1.03 / 1.02 / 1.02 |
//                          0.94 / 1.02 / 1.02 / 1.01
//     bfloat16 1 worker    1.12 / 1.17 / 1.16 / 1.14 | 0.98 / 0.98 / 0.98 / 0.98, 0.96 / 0.95 / 0.98 / 1.01 | 1.00 / 0.98 / 1.00 / 1.01, 1.06 / 1.06 / 1.02 / 1.02 | 0.92 /
//                          1.02 / 1.03 / 1.01
//     bfloat16 8 workers   1.06 / 1.05 / 1.05 / 1.05 | 1.08 / 1.07 / 1.07 / 1.05, 0.97 / 0.96 / 0.98 / 1.00 | 1.04 / 1.03 / 1.03 / 1.03, 1.03 / 1.06 / 1.03 / 1.05 | 0.98 /
//                          1.05 / 1.05 / 1.03
//     tensors around 500 elements, a group each, 82 / 140 / 220 / 320 MiB, bfloat16 4 workers   1.02 / 1.34 / 1.34 / 1.38 | 1.03 / 1.03 / 1.04 / 1.11, 0.96 / 0.95 / 0.93 /
//                          0.97 | 1.01 / 1.01 / 1.00 / 1.04, 1.06 / 1.08 / 1.07 / 1.06 | 1.02 / 1.06 / 1.07 / 1.07
//   PACK, merge arenas of 60 / 120 / 200 / 300 MB together, 150 even tensors, binary32 8 workers: by itself 1.01 / 1.04 / 1.02 / 1.03 | 0.95 / 0.97 / 0.98 / 0.98, a
//   copy of the arenas and reduce_update after it 0.90 / 0.98 / 1.11 / 1.05 | 0.95 / 0.92 / 1.02 / 1.04, reduce_update right after it 0.97 / 0.95 / 0.95 / 0.95 | 0.97 /
//   0.98 / 0.99 / 0.99; tensors around 500 elements, a group each, bfloat16 16 workers: PACK 1.02 / 1.17 / 1.25 / - | 1.01 / 1.00 / 0.99 / 1.00, with the copy
//   1.06 / 1.15 / 1.10 / - | 1.06 / 1.09 / 1.12 / -, without 1.00 / 0.97 / 0.94 / - | 1.04 / 1.02 / 1.02 / -.

// Binary32 launches whose vectors are written through the L2 to memory (agent scope, sc1) as well as streamed (nt): the L2 then does not choose when
// a line leaves it, and the write stream stays in the order of the walk.  Time over streamed alone, models on their lines, 1 / 3 / 4 / 8 / 16 / 32
// workers:
//    66,000 tiles  pipeline 0.991 / 0.987 / 0.989 / 0.988 / 0.987 / 0.991, reduce_update 1.001 / 0.996 / 0.974 / 0.986 / 0.992 / 0.997, direct 1.010 / 0.991 /
//                  0.961 / 0.974 / 0.984 / 0.995
//   200,000 tiles  pipeline 0.976 / 0.981 / 0.993 / 0.980 / 0.984 / 0.988, reduce_update 0.984 / 0.996 / 0.983 / 0.985 / 0.991 / 0.994, direct 0.993 / 0.992 /
//                  0.977 / 0.991 / 0.992 / 0.995
//   500,000 tiles  pipeline 0.971 / 0.985 / 0.988 / 0.989 / 0.996 / 0.997, reduce_update 0.990 / 0.988 / 0.989 / 0.993 / 0.991 / 0.997, direct 0.993 / 0.997 /
//                  0.982 / 0.993 / 0.991 / 0.995; VGG-16 shape, pipeline 0.982 to 0.996 in several runs
// Another card, 65,600 / 80,000 / 100,000 / 150,000 tiles: 1 worker pipeline 0.980 / 0.980 / 0.979 / 0.979, reduce_update 0.991 / 0.984 / 0.988 / 0.994, direct 0.994 /
// 0.983 / 0.988 / 0.993; 2 workers reduce_update 1.000 / 1.006 / 0.997 / 1.002; every other worker count and kind 0.955-1.002.  System scope (sc0 sc1 nt) is the same
// (0.997-1.007); sc1 without nt, in either scope, takes 1.01-1.05 of the time of sc1 nt from 100,000 tiles on.
// The line is the shortest length measured at which nothing is behind: pipeline 30,000 tiles 1.00-1.02.  bfloat16 is level (pipeline 0.995-1.005, reduce_update and direct 0.98-1.01), UPDATE and REDUCE are 0.98-1.01, and PACK
// and models off their lines lose (PACK 1.02-1.08, a thousand small layers 1.02: two tiles write a part of a line each, which the L2 joins).
inline bool goes_through(int kind, int32_t dtype, int32_t tiles, double off_lines, double ragged) {
    if (dtype != MGWFBP_F32 || (kind != K_REDUCE_UPDATE && kind != K_DIRECT && kind != K_PIPELINE)) return false;
    return tiles >= LONG_LAUNCH_TILES / 4 && off_lines <= 0.25 && ragged < 0.025;
}

// What a caller has fixed (mgwfbp_ctx_set_*); the initial values are the library's defaults.
struct LaunchSettings {
    int32_t blocks_per_cu = 0;        // > 0: a persistent grid of that many workgroups per compute unit.  0 = one workgroup
                                      // per unit, dispatched in tile order, which keeps the chip's accesses to each of the
                                      // 2P+2 streams inside a narrow moving window; measured faster for every profile
    int32_t xcd_contiguous = 0;
    int32_t tiles_per_wg = 0;         // 0 = per-kernel default
    int32_t wg_per_cu = 0;            // 0 = per-kernel default, > 0 = cap, < 0 = no cap
    int32_t step_vecs = 0;            // 0 = per-kernel default, > 0 = paced steps, -1 = always the burst form
    int32_t burst_tiles = -1;         // launches of at most this many tiles take the burst form; < 0 = per-kernel default
    uint64_t resident_bytes = 0;      // budget of w + v bytes kept cacheable.  Default none: in a training loop a forward and a
                                      // backward pass run between two updates, so nothing of one is still cached at the next
};

// What the segments [s0, s1) of a launch over `tiles` tiles are like.  Of the launch and not of the model: a large even
// group sent by itself is paced as such whatever the rest of the model looks like.
struct LaunchShares {
    double ragged, off_lines;
};
inline LaunchShares shares_of(const HostTables& h, int32_t s0, int32_t s1, int32_t tiles) {
    const HostTables::SegSums &a = h.seg_sums[static_cast<size_t>(s0)], &b = h.seg_sums[static_cast<size_t>(s1)];
    return {std::min(1.0, static_cast<double>(b.ragged - a.ragged) / tiles),
            b.elems > a.elems ? static_cast<double>(b.off_lines - a.off_lines) / static_cast<double>(b.elems - a.elems) : 0.0};
}

// What a call covers.
struct LaunchWork {
    int kind;
    int32_t dtype, P;
    int32_t tiles;                    // > 0
    double ragged;                    // share of the tiles that are not full or not inside one tensor
    double off_lines;                 // share of the elements of tensors whose tiles start inside the lines of the tensor
    bool reduced;                     // the reduced arena is written
    double resident;                  // share of the tiles whose w and v are kept cacheable
    int32_t segments;
};

struct LaunchShape {
    int32_t tiles_per_wg, units, grid;
    int8_t xcd_contiguous;
    int8_t run_log2;                  // a die's turn is 2^run_log2 consecutive units
    bool may_be_few;                  // the few-segments form may take it
    int form;                         // BURST, PAIRS or the vectors per lane of a paced step
    int32_t wgs_per_cu;               // workgroups that may share a compute unit; <= 0: no cap
    bool rolling;                     // two loads under way in a step (see rolls())
    bool on_lines;                    // steps begin on lines of the weights (see on_lines_pays())
    bool through;                     // vectors are written through the L2 (see goes_through())
    bool in_pieces;                   // ragged tiles piece by piece also where the kernel would rather not (see most_pieces())
};

inline LaunchShape launch_shape(const LaunchSettings& set, const LaunchWork& w, int n_cu) {
    LaunchShape s{};
    // The rules count tiles of 256 elements, the size they were measured with.
    const int32_t length = static_cast<int32_t>(std::min<int64_t>(static_cast<int64_t>(w.tiles) * (TILE / 256), INT32_MAX));
    // A launch too small to fill the chip is bound by the latency of its tiles, not by the memory system: it takes the
    // burst form (every load of a tile at once, no cap) unless the caller has fixed the pacing.
    const bool short_enough = set.burst_tiles < 0 ? length <= default_burst_tiles(w.kind, w.dtype, w.P) : w.tiles <= set.burst_tiles;
    const bool burst = set.step_vecs < 0 || (set.step_vecs == 0 && short_enough);
    // Pairs of tiles: where the rule says so or the caller has asked for several tiles per workgroup, and neither in the
    // burst form, which takes one tile at a time, nor where more than an eighth of the tiles are resident, which are taken
    // one by one (bfloat16, 8 workers, 100,000 tiles: none resident 216 us in pairs against 227 in single tiles, half of
    // them 242 / 213; the lines between cross at 15 %).
    const bool pairs = HAVE_PAIRS && w.kind == K_PIPELINE && w.dtype != MGWFBP_F32 && !burst && w.resident <= 0.125 &&
                       (set.tiles_per_wg > 0 ? set.tiles_per_wg >= PAIR : joined_pipeline(w.dtype, w.P, length, w.ragged));
    const int32_t step = set.step_vecs > 0 ? set.step_vecs : TVECS;
    s.form = burst ? BURST : pairs ? PAIRS : TVECS % 2 == 0 && step >= 2 ? 2 : 1;
    // Tiles per workgroup: PACK runs as single-worker copies, whose tiles are small (one array in, one out), so a
    // workgroup takes several, two at a time; pairs take two at once; every other kind takes one tile
    // per workgroup.  More only stretches the set of bytes the chip has in flight: the window the workgroups of a
    // compute unit cover together should stay within a few hundred KiB per array.
    s.tiles_per_wg = set.tiles_per_wg > 0 ? set.tiles_per_wg
                     : w.kind == K_PACK   ? std::max(1, pack_tiles_per_workgroup(w.dtype, w.P, static_cast<int64_t>(length) * w.P, w.ragged) * 256 / TILE)
                     : pairs              ? PAIR
                                          : 1;
    s.units = (w.tiles + s.tiles_per_wg - 1) / s.tiles_per_wg;
    s.grid = s.units;
    if (set.blocks_per_cu > 0 && n_cu > 0 && static_cast<int64_t>(n_cu) * set.blocks_per_cu < s.units)
        s.grid = n_cu * set.blocks_per_cu;
    if (set.xcd_contiguous && s.grid >= 64) {
        s.grid &= ~7;
        s.xcd_contiguous = 1;
    }
    const int compute_units = n_cu > 0 ? n_cu : 256;
    const int32_t per_cu = (s.units + compute_units - 1) / compute_units;
    // The few-segments form has no tile headers, so it serves neither the resident share of w and v, which they
    // mark, nor the forms in which a workgroup goes on to tiles far from its first.
    const bool one_turn = s.grid == s.units && !s.xcd_contiguous;
    s.may_be_few = HAVE_FEW && one_turn && !(updates(w.kind) && set.resident_bytes > 0) && (w.segments <= FEW || !needs_owner(w.kind)) &&
                   few_form_pays(w.kind, w.dtype, w.P, length, w.segments, per_cu);
    // Forms of long launches, in the table form only.
    s.on_lines = HAVE_PIECES && s.form == 1 && on_lines_pays(w.kind, w.dtype, w.reduced, length, w.segments, w.off_lines);
    if (s.on_lines) s.may_be_few = false;
    s.through = s.form == 1 && !s.may_be_few && !s.on_lines && goes_through(w.kind, w.dtype, length, w.off_lines, w.ragged);
    // With the form, the workgroups that may share a compute unit set the loads it has in flight (1 KiB of a binary32 array
    // per vector of a step and workgroup, half that of a 16-bit one).
    s.wgs_per_cu = set.wg_per_cu;
    if (s.wgs_per_cu == 0) {
        s.wgs_per_cu = burst ? -1 : default_workgroups_per_cu(w.kind, w.dtype, w.P, length, w.ragged, w.reduced, s.form);
        if (s.form == PAIRS ? length < 2 * SHORT_LAUNCH_TILES : w.dtype == MGWFBP_F32 && w.kind != K_PACK && few_rounds(length, w.P))
            s.wgs_per_cu = short_launch_cap(s.wgs_per_cu, w.kind, w.P, s.may_be_few && s.form != PAIRS, per_cu);
        if (s.wgs_per_cu <= 0 && w.ragged <= 0.25 && even_rounds(w.kind, w.dtype, w.P, s.may_be_few, s.form, per_cu)) s.wgs_per_cu = 25;
    }
    s.rolling = may_roll(w.kind, s.form) && set.step_vecs == 0 && set.wg_per_cu == 0 && rolls(w.dtype, w.P, s.may_be_few, per_cu);
    s.in_pieces = w.ragged > 0.5;
    s.run_log2 = one_turn && (!s.on_lines || (w.resident == 0 && runs_on_lines(w.kind, w.dtype, w.P, length, w.segments))) ? run_log2_of(w.kind, w.dtype, w.P, w.off_lines) : int8_t{0};
    return s;
}

}  // namespace

#endif
