// Device side of the MG-WFBP library for gfx950 (MI355X): context management and the streaming
// kernels pack / reduce / unpack_update and their fused forms.
//
// All six operations are the same walk over the merge arena, tile by tile (by default one workgroup
// of 64 lanes = one wavefront per tile of 256 elements, dispatched in tile order):
//
//   kind            reads                          writes
//   PACK            per-layer gradients (P)        merge arenas (P)                     Sec. 5.3
//   REDUCE          merge arenas (P)               reduced arena                        Eq. 2 (sum, 1/P)
//   UPDATE          reduced arena, w, v            w, v                                 Eq. 2 (update)
//   REDUCE_UPDATE   merge arenas (P), w, v         w, v
//   PIPELINE        per-layer gradients (P), w, v  merge arenas (P), [reduced], w, v
//   DIRECT          per-layer gradients (P), w, v  [reduced], w, v
//
// The arena side of an access is 16-byte aligned in full tiles (they start on multiples of the tile size and
// lanes step in 4-element vectors) and starts on any element in ragged ones.  The per-layer side starts wherever the
// tensor starts.  So both are accessed through vector types that only promise element alignment; gfx950 executes those as
// the same 16-byte (8-byte for 16-bit gradients) memory instructions.
//
// A tile that lies entirely inside one tensor takes the fast path: tensor index and source offset
// come from the tile header, the pointer table is read once with wave-uniform addresses, and the tile is
// walked in paced steps, one worker at a time (see paced_step).  Any other tile that holds a few pieces of tensors (nearly
// always one: the end of a group) is taken piece by piece (one_piece, several_pieces).  What is left takes the general path:
// the tile-local start offsets of the segments it intersects are produced by a workgroup-wide prefix sum
// (wavefront scans via cross-lane shifts, combined through LDS) over the segment lengths, staged in LDS,
// and each lane finds the owner of its vector by binary search there.  Vectors that straddle two tensors,
// the end of the group or the edge of the interval a call is clipped to are taken element by element,
// one element per lane, after the whole vectors.
//
// A launch over at most eight segments (one group, a tensor that has just arrived) takes a second form of the kernel
// that gets the segments as arguments and reads no tables (mgwfbp_few_kernel).
//
// This is bandwidth-bound streaming work (at most 4 flops per 12+ bytes), so there is no use for the
// matrix cores; the job is to present the traffic to the memory system in the form it serves fastest:
//   - SMALL LAUNCHES (too few tiles to fill the chip: one small group) are bound by the latency of a tile,
//     so they issue every load of a tile at once (the burst form); what follows is for the rest;
//   - PACING.  For these read/write mixes MI355X delivers most when every compute unit keeps about
//     16-24 KiB of loads in flight and a tenth less beyond that, so a lane has one 16-byte load outstanding
//     (one worker's share of the tile; two workers' in the kinds that only read between their stores, and in the
//     pipeline's launches whose wavefronts are few or have little under way, see rolls()) and each
//     launch asks for enough unused LDS that only so many workgroups share a compute unit, 12 to 25 or all of them
//     by kind, gradient width, worker count, length and what the launch covers (the rules are in launch.h);
//   - SMALL WORKGROUPS.  A workgroup is one wavefront and a tile the 256 elements it covers with one vector per
//     lane: the same bytes in flight spread over sixteen independent wavefronts per compute unit, each at its
//     own point of its walk, load the memory system more evenly than two workgroups of four wavefronts that
//     move in step (3-5 % of the peak on every shape);
//   - one workgroup per tile, dispatched in tile order, so that the bytes the chip has in flight form one
//     contiguous moving window per array; where tiles start inside the lines of their tensors, runs of a few tiles
//     per die inside that window (unit_of());
//   - 16-BIT GRADIENTS: a long pipeline launch takes two tiles per workgroup, 16 bytes of gradients per lane, so
//     that a wavefront has as much under way as with binary32 (joined_tiles);
//   - everything is streamed with non-temporal loads and stores (long binary32 launches also write through the L2, goes_through());
//     a caller may ask for a leading share of the weights and momenta to use ordinary accesses and stay in the 256 MB memory-side
//     cache (tile flag);
//   - PACK, which has no arithmetic across workers, runs as P single-worker copies (gridDim.y = P),
//     so the chip streams 2 arrays at a time instead of 2P; a workgroup copies 1 to 4 KiB of its worker's data,
//     two tiles per step (more per workgroup stretches the window its compute unit covers and costs 8 %).
//
// Arithmetic contract: binary32, one rounding per operation.  The file must be compiled with
// -ffp-contract=off so that mu*v + g and w - lr*v are never fused.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <chrono>
#include <cmath>
#include <cstddef>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <type_traits>

#include "launch.h"
#include "mgwfbp.h"
#include "tables.h"

#ifndef MGWFBP_NT
#define MGWFBP_NT 3   // bit 0: non-temporal loads of gradients / merge / reduced, bit 1: non-temporal
                      // stores to merge / reduced, bit 2: non-temporal accesses to w and v
#endif

// Table space of mgwfbp_group_pipeline_static: one copy per GPU, held until the process ends.  Host code must
// not pass this name to a kernel or a copy (on the host it is only a stand-in for the symbol); the device
// address comes from hipGetSymbolAddress, once per device.  (No `used` attribute here: the compiler exports a
// file-local device variable under a global symbol only when it sees host code refer to it, as
// mgwfbp_group_pipeline_static does; marked `used` it stays a local symbol that the runtime cannot look up.)
static __device__ __align__(256) unsigned char scratch[MGWFBP_STATIC_TABLE_MAX_BYTES];

namespace {

// ---------------------------------------------------------------------------------------------
// vector types that promise only element alignment
// ---------------------------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4), aligned(2)));   // bfloat16 bit patterns
typedef _Float16 f16x4 __attribute__((ext_vector_type(4), aligned(2)));   // IEEE binary16

typedef uint16_t u16x8 __attribute__((ext_vector_type(8), aligned(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8), aligned(2)));

template <typename T, int W> struct VecOf;
template <> struct VecOf<float, 4> { typedef f32x4 type; };
template <> struct VecOf<float, 1> { typedef float type; };
template <> struct VecOf<uint16_t, 4> { typedef u16x4 type; };
template <> struct VecOf<uint16_t, 8> { typedef u16x8 type; };
template <> struct VecOf<_Float16, 8> { typedef f16x8 type; };
template <> struct VecOf<uint16_t, 1> { typedef uint16_t type; };
template <> struct VecOf<_Float16, 4> { typedef f16x4 type; };
template <> struct VecOf<_Float16, 1> { typedef _Float16 type; };

template <typename V> struct Lanes { static constexpr int n = 4; };
template <> struct Lanes<float> { static constexpr int n = 1; };
template <> struct Lanes<uint16_t> { static constexpr int n = 1; };
template <> struct Lanes<_Float16> { static constexpr int n = 1; };

__device__ __forceinline__ float comp(const f32x4& v, int c) { return v[c]; }
__device__ __forceinline__ float comp(const float& v, int) { return v; }
__device__ __forceinline__ uint16_t comp(const u16x4& v, int c) { return v[c]; }
__device__ __forceinline__ uint16_t comp(const uint16_t& v, int) { return v; }
__device__ __forceinline__ _Float16 comp(const f16x4& v, int c) { return v[c]; }
__device__ __forceinline__ _Float16 comp(const _Float16& v, int) { return v; }
__device__ __forceinline__ void setc(f32x4& v, int c, float x) { v[c] = x; }
__device__ __forceinline__ void setc(float& v, int, float x) { v = x; }

// Address spaces of the AMDGPU target: 1 = global memory, 4 = constant (read-only for the whole
// kernel; wave-uniform addresses are fetched through the scalar unit).  Pointers that were themselves
// read from memory carry no address space, so data accesses name it explicitly; otherwise they would
// become slower generic ("flat") instructions.
#define MGWFBP_GLOBAL __attribute__((address_space(1)))
#define MGWFBP_CONST __attribute__((address_space(4)))

template <typename T> __device__ __forceinline__ const MGWFBP_CONST T* ro(const T* p) {
    return (const MGWFBP_CONST T*)p;
}

template <bool NT, typename V> __device__ __forceinline__ V ld(const void* p) {
    const MGWFBP_GLOBAL V* q = (const MGWFBP_GLOBAL V*)p;
    if constexpr (NT) return __builtin_nontemporal_load(q);
    else return *q;
}
// THROUGH_L2: 16-byte vectors are written through the L2 (sc1: agent scope) as well as streamed.  There is no builtin for that on vectors.  The no-op
// is the two wait states gfx950 wants between a store of more than 8 bytes and the next write of its registers, which the compiler
// sees to after the stores it knows.
template <bool NT, typename V, bool THROUGH_L2 = false> __device__ __forceinline__ void st(void* p, const V& x) {
    MGWFBP_GLOBAL V* q = (MGWFBP_GLOBAL V*)p;
    if constexpr (NT && THROUGH_L2 && sizeof(V) == 16) asm volatile("global_store_dwordx4 %0, %1, off sc1 nt\n\ts_nop 1" ::"v"(q), "v"(x) : "memory");
    else if constexpr (NT) __builtin_nontemporal_store(x, q);
    else *q = x;
}

constexpr bool NT_LD = (MGWFBP_NT & 1) != 0;
constexpr bool NT_ST = (MGWFBP_NT & 2) != 0;
constexpr bool NT_WV = (MGWFBP_NT & 4) != 0;

__device__ __forceinline__ float widen(float x) { return x; }
__device__ __forceinline__ float widen(uint16_t bits) { return __uint_as_float(static_cast<uint32_t>(bits) << 16); }
__device__ __forceinline__ float widen(_Float16 x) { return static_cast<float>(x); }   // every binary16 value is a binary32 value

// ---------------------------------------------------------------------------------------------
// kernel arguments
// ---------------------------------------------------------------------------------------------
//
// What a launch costs the host depends on the size of this block: up to 112 bytes a launch takes 2.5 us (1.35 without any
// argument), from 136 bytes on 3.3 us (the runtime writes the block into device memory and reads back from it before it rings
// the doorbell), and a kernel that asks for gridDim makes the runtime append 256 more.  So everything that can be derived from something else is, and the grid
// size that the persistent form needs comes in as `turn`.
constexpr int XCD_CONTIGUOUS = 1, ROLLING = 2, IN_PIECES = 4;
template <typename GradT> struct CallArgs {
    const GradT* const* grad_ptrs;   // [P*L]
    GradT* const* merge_bufs;        // [P]
    float* reduced;                  // arena or null
    float* const* w_ptrs;            // [L]
    float* const* v_ptrs;            // [L]
    float lr, mu, inv_p;
    int32_t L, P;
    int32_t tile_first, tile_count;
    int16_t tiles_per_wg;            // consecutive tiles one workgroup handles per turn, >= 1
    int8_t flags;                    // XCD_CONTIGUOUS, ROLLING, IN_PIECES
    int8_t run_log2;                 // a die's turn is 2^run_log2 consecutive units, see unit_of()
};
template <typename GradT> struct Args : CallArgs<GradT> {      // table form: what a tile holds is in the tables
    const TileHdr* tiles;            // the segment tables lie right below, see seg_tables()
    int32_t n_seg;                   // segments of the model
    int32_t n_units;                 // ceil(tile_count / tiles_per_wg)
    int32_t turn;                    // units from one of a workgroup's turns to its next: the workgroups of a walk
    int16_t clip_lo, clip_hi;        // first element wanted of the first tile, end of those wanted of the last one
};
template <typename GradT> struct FewArgs : CallArgs<GradT> {   // few-segments form: the segments come along
    int32_t layer_hi;                // tensor of segment 0; segment j is tensor layer_hi - j
    int16_t start0;                  // first element of segment 0; all positions count from the first tile's start
    uint8_t n;                       // segments, 1..FEW
    uint8_t closes;                  // bit j: segment j ends its group, the next one starts on the next tile
    int32_t end[FEW];                // end of segment j
};
static_assert(sizeof(Args<float>) <= 112 && sizeof(FewArgs<float>) <= 112,
              "a larger block of arguments makes every launch 0.9 us dearer");

// Unit a workgroup starts with.  Workgroups are dealt round-robin to the 8 dies, each with an L2 of its own, so in
// plain order neighbouring tiles belong to different dies.  Where tiles do not start on the 128-byte lines of the
// tensors, two dies then fetch the line they share.  Runs of a few consecutive units per die (within every 8 runs of
// the dispatch order, so that the chip still moves through one window) let all but one boundary of a run meet in one L2
// (bytes the L2s fetch over those needed, 300 views of odd sizes, 8 workers: pipeline 1.139 -> 1.046, update 1.126 ->
// 1.036, direct 1.138 -> 1.030; what they write stays at 1.01-1.04).  GB/s, 300 tensors of odd sizes around 100,000 elements as views of
// flat buffers, 8 workers, runs of 1 / 4 / 8 / 16: direct bf16 5144 / 5716 / 5885 / 5937, unpack_update 5514 / 6042 /
// 6085 / 6185, pipeline f32 5613 / 5888 / 5748 / 5664; on the ResNet-50 shape, nearly all of whose tiles start on lines:
// pipeline f32 6224 / 6131 / 6005 / 5835, unpack_update 6468 / 6326 / 6344 / 6221.
template <typename GradT> __device__ __forceinline__ int unit_of(const CallArgs<GradT>& A) {
    const int b = static_cast<int>(blockIdx.x);
    const int r = A.run_log2;
    if (r == 0) return b;
    const int within = b & ((8 << r) - 1);
    const int last = b - within + (8 << r) - 1;           // last unit of this set of eight runs
    if (static_cast<int64_t>(last) * A.tiles_per_wg >= A.tile_count) return b;      // the launch ends before it
    return b - within + ((within & 7) << r) + (within >> 3);
}

// What a path works out from x stays on that path.  The compiler moves whatever does not change from tile to tile in front
// of the walk, where every workgroup pays for it: lane masks of the prefix sum, addresses of the segment tables and starts of
// the segments of the few-segments form were some 100 instructions in front of tiles that need none of them, and a dozen
// registers.  With the arguments fetched in one trip (see the kernels) a launch of 1 to 1000 tiles takes 0.1-0.5 us less: 10 tiles and
// a ragged one, 8 workers, pipeline 2.32 -> 2.16, pack 1.97 -> 1.84, unpack_update 2.06 -> 1.87; 1000 tiles, unpack_update 3.22 -> 2.67.
__device__ __forceinline__ void here_only(int32_t& x) { asm volatile("" : "+s"(x)); }          // the same for all lanes
__device__ __forceinline__ void here_only_per_lane(int32_t& x) { asm volatile("" : "+v"(x)); }

// The tables of one model lie in one block: seg_layer[S], seg_n[S] and seg_off[S + 1], ending where the tile headers
// begin, so that the address of the headers and S lead to all of them.
struct SegTables {
    const uint64_t* off;
    const uint32_t* n;
    const int32_t* layer;
};
template <typename GradT> __device__ __forceinline__ SegTables seg_tables(const Args<GradT>& A) {
    int32_t S = A.n_seg;
    here_only(S);
    SegTables t;
    t.off = reinterpret_cast<const uint64_t*>(A.tiles) - (S + 1);
    t.n = reinterpret_cast<const uint32_t*>(t.off) - S;
    t.layer = reinterpret_cast<const int32_t*>(t.n) - S;
    return t;
}

// First worker a workgroup serves.  PACK has no arithmetic across workers, so it is launched as P
// single-worker copies side by side in gridDim.y: workgroups are dispatched x-fastest, the chip then
// streams one worker's gradients at a time (2 streams instead of 2P), which the memory system serves
// faster.
template <int KIND> __device__ __forceinline__ int worker_base() {
    return KIND == K_PACK ? static_cast<int>(blockIdx.y) : 0;
}

// Pointers of the P workers, either held in registers (P known at compile time) or re-read from the
// table on every use (any P).
template <typename T, int PT> struct WorkerPtrs {
    T* p[PT];
    __device__ __forceinline__ void fetch(T* const* table, int64_t stride, int64_t index, int w0) {
#pragma unroll
        for (int w = 0; w < PT; ++w) p[w] = ro(table)[(w0 + w) * stride + index];
    }
    __device__ __forceinline__ T* get(int w) const { return p[w]; }
};
template <typename T> struct WorkerPtrs<T, 0> {
    T* const* base;
    int64_t stride;
    __device__ __forceinline__ void fetch(T* const* table, int64_t s, int64_t index, int w0) {
        base = table + w0 * s + index;
        stride = s;
    }
    __device__ __forceinline__ T* get(int w) const { return ro(base)[w * stride]; }
};

// ---------------------------------------------------------------------------------------------
// one paced step: N vectors (W = 4) or one element (W = 1) per lane, at arena position `apos`, which is
// element `soff` of its tensor; the N vectors lie `stride` elements apart
// ---------------------------------------------------------------------------------------------
//
// The step is taken worker by worker: load one worker's values, store them into that worker's merge arena
// (kinds that fill the arenas), add them to the running sums -- acc = g_0, then acc = acc + g_w, the worker
// order 0..P-1 of Eq. 2 -- and go on to the next worker; then the reduced arena, then v, then w.  A lane never
// has more than N loads in flight (kinds without stores between the workers take MGWFBP_READ_GROUP workers at a
// time), and that is the point: the memory system serves this traffic fastest when each compute unit keeps
// only 16-24 KiB of loads in flight (the exact figure differs a little from one machine to the next) and about
// a tenth slower beyond.  N x 16 bytes per lane of the workgroup times the workgroups a compute unit is allowed
// to hold (see launch.h) sets that budget.
#ifndef MGWFBP_READ_GROUP
#define MGWFBP_READ_GROUP 2
#endif
// Workers whose loads go out together in the burst form and in ragged tiles where the worker count is not compiled (where it
// is: all of them).  us with four / eight, 12 tensors of one group, 300 and 1100 tiles, binary32: pipeline 5 workers 4.8 / 4.3, 7.4 / 6.4; 12
// workers 7.7 / 6.6, 10.9 / 9.6; 32 workers 15.8 / 11.0, 23.7 / 19.2; direct 32 workers 14.1 / 9.6, 17.2 / 12.6.  The longest launches of the burst
// form would rather have four: 150 equal tensors, binary32, 1650 tiles, 32 workers reduce 10.9 / 11.4, reduce_update 12.0 / 12.7; bfloat16
// pipeline, 12 workers, 3000 tiles 10.7 / 11.3; three of three at once binary32, 3000 tiles 6.5 / 7.0.
#ifndef MGWFBP_TOGETHER
#define MGWFBP_TOGETHER 8
#endif
#ifndef MGWFBP_GENERAL_GROUP
#define MGWFBP_GENERAL_GROUP 64   // workers whose loads ragged tiles issue together where the count is compiled (64: all of them)
#endif

// keeps the compiler from moving the next group's loads above this group's arithmetic
__device__ __forceinline__ void pace() { __builtin_amdgcn_sched_barrier(0); }

// the last part of a paced step: v, then w
template <int N, bool WVNT, bool THROUGH_L2, typename GradT, typename FV>
__device__ __forceinline__ void update_step(const CallArgs<GradT>& A, float* wp, float* vp, int64_t soff, int stride,
                                            const FV* acc) {
    constexpr int C = Lanes<FV>::n;
    FV v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = ld<WVNT, FV>(vp + soff + i * stride);
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float t1 = A.mu * comp(v[i], c);
            setc(v[i], c, t1 + comp(acc[i], c));
        }
        st<WVNT, FV, THROUGH_L2>(vp + soff + i * stride, v[i]);
    }
    pace();
    FV w[N];
#pragma unroll
    for (int i = 0; i < N; ++i) w[i] = ld<WVNT, FV>(wp + soff + i * stride);
#pragma unroll
    for (int i = 0; i < N; ++i) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float t2 = A.lr * comp(v[i], c);
            setc(w[i], c, comp(w[i], c) - t2);
        }
        st<WVNT, FV, THROUGH_L2>(wp + soff + i * stride, w[i]);
    }
}

template <int N> struct Int { static constexpr int value = N; };
// f(Int<n>()) for an n of 1 .. MOST; nothing for 0.
template <int MOST, typename F> __device__ __forceinline__ void some_sizes(int n, F&& f) {
    if constexpr (MOST > 0) {
        if (n == MOST) f(Int<MOST>());
        else some_sizes<MOST - 1>(n, f);
    }
}

template <int KIND, typename GradT, int PT, int W, int N, bool WVNT, int TOGETHER = 0, int GENERAL = MGWFBP_GENERAL_GROUP>
__device__ __forceinline__ void paced_step(const CallArgs<GradT>& A, const WorkerPtrs<const GradT, PT>& src,
                                           const WorkerPtrs<GradT, PT>& mrg, float* wp, float* vp,
                                           int64_t soff, int64_t apos, int stride) {
    typedef typename VecOf<GradT, W>::type GV;
    typedef typename VecOf<float, W>::type FV;
    constexpr int C = Lanes<GV>::n;
    FV acc[N];
    // the burst form and ragged tiles want everything under way at once: their v and w loads go out before the gradients'
    constexpr int NE = (updates(KIND) && TOGETHER > 0) ? N : 1;
    FV v_early[NE], w_early[NE];
    if constexpr (updates(KIND) && TOGETHER > 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) v_early[i] = ld<WVNT, FV>(vp + soff + i * stride);
#pragma unroll
        for (int i = 0; i < N; ++i) w_early[i] = ld<WVNT, FV>(wp + soff + i * stride);
    }
    if constexpr (reads_grads(KIND) || reads_merge(KIND)) {
        // workers whose loads are issued together: one (kinds that store each worker's share before the next
        // load), MGWFBP_READ_GROUP (kinds that only read them), or all of them / TOGETHER at a time (the burst form and
        // the ragged tiles, whose time is the chain of trips to memory)
        constexpr int GW = TOGETHER > 0 ? (PT > 0 ? (PT < GENERAL ? PT : GENERAL) : TOGETHER) : (writes_merge(KIND) ? 1 : MGWFBP_READ_GROUP);
        auto some_workers = [&](auto size, int w0) {      // workers w0 .. w0 + size - 1
            constexpr int COUNT = decltype(size)::value;
            GV g[COUNT][N];
#pragma unroll
            for (int j = 0; j < COUNT; ++j) {
                const GradT* from;
                if constexpr (reads_grads(KIND)) from = src.get(w0 + j) + soff;
                else from = mrg.get(w0 + j) + apos;
#pragma unroll
                for (int i = 0; i < N; ++i) g[j][i] = ld<NT_LD, GV>(from + i * stride);
            }
            // every load of the group is issued before the first value is used (left alone, the scheduler now and then puts
            // an add, and with it a wait for the first load, in front of the second load); with a compiled worker count the
            // kinds that do not store each worker's share want the groups to run into one another instead
            if constexpr ((writes_merge(KIND) && sums(KIND)) || PT == 0) pace();
#pragma unroll
            for (int j = 0; j < COUNT; ++j) {
                if constexpr (writes_merge(KIND)) {
                    GradT* to = mrg.get(w0 + j) + apos;
#pragma unroll
                    for (int i = 0; i < N; ++i) st<NT_ST, GV, through(KIND)>(to + i * stride, g[j][i]);
                }
                if constexpr (sums(KIND)) {
#pragma unroll
                    for (int i = 0; i < N; ++i)
#pragma unroll
                        for (int c = 0; c < C; ++c) {
                            const float x = widen(comp(g[j][i], c));
                            setc(acc[i], c, (w0 + j == 0) ? x : comp(acc[i], c) + x);
                        }
                }
            }
            pace();
        };
        if constexpr (PT > 0) {
#pragma unroll
            for (int w0 = 0; w0 < PT; w0 += GW) {
                if (w0 + GW <= PT) some_workers(Int<GW>(), w0);
                else some_workers(Int<PT % GW + (PT % GW == 0)>(), w0);
            }
        } else {
            // A worker count that is not compiled: whole groups, then one of the size that is left, so that no worker
            // costs a branch and none waits for another group that it could have been part of.
            int w0 = 0;
            for (; w0 + GW <= A.P; w0 += GW) some_workers(Int<GW>(), w0);
            some_sizes<GW - 1>(A.P - w0, [&](auto size) { some_workers(size, w0); });
        }
        if constexpr (sums(KIND)) {
#pragma unroll
            for (int i = 0; i < N; ++i)
#pragma unroll
                for (int c = 0; c < C; ++c) setc(acc[i], c, comp(acc[i], c) * A.inv_p);
        }
    }
    if constexpr (KIND == K_UPDATE) {
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = ld<NT_LD, FV>(A.reduced + apos + i * stride);
    }
    if constexpr (writes_reduced(KIND)) {
        if (KIND == K_REDUCE || A.reduced != nullptr) {
#pragma unroll
            for (int i = 0; i < N; ++i) st<NT_ST, FV, through(KIND)>(A.reduced + apos + i * stride, acc[i]);
        }
    }
    if constexpr (updates(KIND) && TOGETHER > 0) {              // (never through the L2: a launch that is has few ragged tiles)
#pragma unroll
        for (int i = 0; i < N; ++i) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const float t1 = A.mu * comp(v_early[i], c);
                setc(v_early[i], c, t1 + comp(acc[i], c));
                const float t2 = A.lr * comp(v_early[i], c);
                setc(w_early[i], c, comp(w_early[i], c) - t2);
            }
            st<WVNT, FV>(vp + soff + i * stride, v_early[i]);
            st<WVNT, FV>(wp + soff + i * stride, w_early[i]);
        }
    } else if constexpr (updates(KIND)) {
        update_step<N, WVNT, through(KIND)>(A, wp, vp, soff, stride, acc);
    }
}
// one vector or element of the general path
template <int KIND, typename GradT, int PT, int W>
__device__ __forceinline__ void do_one(const CallArgs<GradT>& A, const WorkerPtrs<GradT, PT>& mrg,
                                       int layer, int64_t soff, int64_t apos) {
    WorkerPtrs<const GradT, PT> src;
    float* wp = nullptr;
    float* vp = nullptr;
    if constexpr (reads_grads(KIND)) src.fetch(A.grad_ptrs, A.L, layer, worker_base<KIND>());
    if constexpr (updates(KIND)) {
        wp = ro(A.w_ptrs)[layer];
        vp = ro(A.v_ptrs)[layer];
    }
    paced_step<KIND, GradT, PT, W, 1, NT_WV, MGWFBP_TOGETHER>(A, src, mrg, wp, vp, soff, apos, 0);
}

// ---------------------------------------------------------------------------------------------
// fast path: `nvec` vectors per lane (one or more whole tiles) that lie inside one tensor, taken STEPV
// vectors at a time; vector u of the chunk covers elements u * BLOCK * VEC + lane * VEC ...
// ---------------------------------------------------------------------------------------------
template <int KIND, typename GradT, int PT, bool WVNT, int STEPV>
__device__ __forceinline__ void fast_chunk(const CallArgs<GradT>& A, const WorkerPtrs<GradT, PT>& mrg,
                                           int layer, int64_t tensor_off, int64_t tile_base, int nvec) {
    static_assert(STEPV == 0 || TVECS % STEPV == 0, "a tile is a whole number of steps");
    WorkerPtrs<const GradT, PT> src;
    float* wp = nullptr;
    float* vp = nullptr;
    if constexpr (reads_grads(KIND)) src.fetch(A.grad_ptrs, A.L, layer, worker_base<KIND>());
    if constexpr (updates(KIND)) {
        wp = ro(A.w_ptrs)[layer];
        vp = ro(A.v_ptrs)[layer];
    }
    constexpr int STEP = BLOCK * VEC;
    int lane_elem = static_cast<int>(threadIdx.x) * VEC;
    // Left alone, the compiler sets up every arena's address plus this in front of the walk, two registers per worker: 138 for
    // binary32 reductions of 16 workers instead of 70 (4000 tiles over 150 tensors 17.0 us, so 12.5).  A direct step has no arenas, and is
    // faster as the compiler has it (bfloat16, 16 workers, 12,000 tiles 24.3 us, so 25.3).
    if constexpr (!directs(KIND)) here_only_per_lane(lane_elem);
    const int64_t soff = tensor_off + lane_elem;    // this lane's first element: in its tensor
    const int64_t apos = tile_base + lane_elem;     //                            in the arena
    if constexpr (STEPV == 0) {
        // burst: every load of the tile under way at once.  The form for a launch too small to fill the chip,
        // where the time is the tile's own latency and not the memory system's throughput.  (Of builds that do not take
        // tiles in pieces: the others take a full tile in the burst form as one piece.)
        for (int u = 0; u < nvec; u += TVECS)
            paced_step<KIND, GradT, PT, VEC, TVECS, WVNT, MGWFBP_TOGETHER>(A, src, mrg, wp, vp,
                                                                soff + static_cast<int64_t>(u) * STEP,
                                                                apos + static_cast<int64_t>(u) * STEP, STEP);
    } else {
        for (int u = 0; u < nvec; u += STEPV) {
            paced_step<KIND, GradT, PT, VEC, STEPV, WVNT>(A, src, mrg, wp, vp, soff + static_cast<int64_t>(u) * STEP,
                                                          apos + static_cast<int64_t>(u) * STEP, STEP);
            pace();
        }
    }
}

// Several full tiles of one tensor in one step (see joined_tiles_of()).
constexpr int WIDE = 8;               // 16-bit gradients per lane in a joined pipeline step: 16 bytes

template <int KIND, typename GradT, int PT>
__device__ __forceinline__ void joined_tiles(const CallArgs<GradT>& A, const WorkerPtrs<GradT, PT>& mrg, int layer,
                                             int64_t tensor_off, int64_t tile_base, float* s_sums) {
    WorkerPtrs<const GradT, PT> src;
    src.fetch(A.grad_ptrs, A.L, layer, worker_base<KIND>());
    int lane_elem = static_cast<int>(threadIdx.x) * VEC;
    here_only_per_lane(lane_elem);
    if constexpr (KIND == K_PACK) {
        paced_step<KIND, GradT, PT, VEC, PACK_TILES * TVECS, true>(A, src, mrg, nullptr, nullptr, tensor_off + lane_elem,
                                                             tile_base + lane_elem, BLOCK * VEC);
    } else {
        // One worker at a time as in paced_step, with 16 bytes per lane, 8 consecutive elements: a worker's share
        // is the 1 KiB it is with binary32.  The sums then change hands through LDS, so that the binary32 arrays,
        // too, are accessed with consecutive 16 bytes per lane.
        static_assert(PAIRED == BLOCK * WIDE, "16 bytes per lane");
        typedef typename VecOf<GradT, WIDE>::type GV;
        constexpr int N = PAIRED / (BLOCK * VEC);
        float* wp = ro(A.w_ptrs)[layer];
        float* vp = ro(A.v_ptrs)[layer];
        const int wide_elem = static_cast<int>(threadIdx.x) * WIDE;
        float sum[WIDE];
        auto worker = [&](int w) {
            const GV g = ld<NT_LD, GV>(src.get(w) + tensor_off + wide_elem);
            pace();
            st<NT_ST, GV>(mrg.get(w) + tile_base + wide_elem, g);
#pragma unroll
            for (int e = 0; e < WIDE; ++e) {
                const float x = widen(static_cast<GradT>(g[e]));
                sum[e] = w == 0 ? x : sum[e] + x;
            }
            pace();
        };
        if constexpr (PT > 0) {
#pragma unroll
            for (int w = 0; w < PT; ++w) worker(w);
        } else {
            for (int w = 0; w < A.P; ++w) worker(w);
        }
        __syncthreads();                       // the previous step's readers are done with LDS
#pragma unroll
        for (int e = 0; e < WIDE; ++e) s_sums[wide_elem + e] = sum[e] * A.inv_p;
        __syncthreads();
        f32x4 acc[N];
#pragma unroll
        for (int i = 0; i < N; ++i) acc[i] = *reinterpret_cast<const f32x4*>(s_sums + lane_elem + i * BLOCK * VEC);
        if (A.reduced != nullptr) {
#pragma unroll
            for (int i = 0; i < N; ++i) st<NT_ST, f32x4>(A.reduced + tile_base + lane_elem + i * BLOCK * VEC, acc[i]);
        }
        update_step<N, true, false>(A, wp, vp, tensor_off + lane_elem, BLOCK * VEC, acc);
    }
}

// ---------------------------------------------------------------------------------------------
// rolling steps of the pipeline
// ---------------------------------------------------------------------------------------------
//
// A tile of the pipeline with two loads under way instead of one: the next worker's goes out before this one's is stored,
// and v and w follow the last worker's.  For the launches whose wavefronts are too few, or too narrow, to keep enough under
// way with one each (see rolls()).
template <typename GradT, int PT>
__device__ __forceinline__ void rolling_tile(const CallArgs<GradT>& A, const WorkerPtrs<GradT, PT>& mrg, int layer, int64_t tensor_off,
                                             int64_t tile_base) {
    typedef typename VecOf<GradT, VEC>::type GV;
    WorkerPtrs<const GradT, PT> src;
    src.fetch(A.grad_ptrs, A.L, layer, 0);
    float* wp = ro(A.w_ptrs)[layer];
    float* vp = ro(A.v_ptrs)[layer];
    int lane_elem = static_cast<int>(threadIdx.x) * VEC;
    here_only_per_lane(lane_elem);
    const int64_t soff = tensor_off + lane_elem, apos = tile_base + lane_elem;
    f32x4 acc;
    auto load = [&](int k) {
        const GV g = ld<NT_LD, GV>(src.get(k) + soff);
        pace();
        return g;
    };
    auto use = [&](const GV& g, int k) {
        st<NT_ST, GV>(mrg.get(k) + apos, g);
#pragma unroll
        for (int c = 0; c < VEC; ++c) {
            const float x = widen(comp(g, c));
            setc(acc, c, k == 0 ? x : comp(acc, c) + x);
        }
        pace();
    };
    GV g = load(0);
    if constexpr (PT > 0) {
#pragma unroll
        for (int k = 0; k + 1 < PT; ++k) {
            const GV next = load(k + 1);
            use(g, k);
            g = next;
        }
    } else {
        for (int k = 0; k + 1 < A.P; ++k) {
            const GV next = load(k + 1);
            use(g, k);
            g = next;
        }
    }
    f32x4 v = ld<true, f32x4>(vp + soff);
    pace();
    use(g, (PT > 0 ? PT : A.P) - 1);
    f32x4 w = ld<true, f32x4>(wp + soff);
    pace();
#pragma unroll
    for (int c = 0; c < VEC; ++c) setc(acc, c, comp(acc, c) * A.inv_p);
    if (A.reduced != nullptr) st<NT_ST, f32x4>(A.reduced + apos, acc);
#pragma unroll
    for (int c = 0; c < VEC; ++c) {
        const float t1 = A.mu * comp(v, c);
        setc(v, c, t1 + comp(acc, c));
    }
    st<true, f32x4>(vp + soff, v);
    pace();
#pragma unroll
    for (int c = 0; c < VEC; ++c) {
        const float t2 = A.lr * comp(v, c);
        setc(w, c, comp(w, c) - t2);
    }
    st<true, f32x4>(wp + soff, w);
}

// ---------------------------------------------------------------------------------------------
// ragged tiles: a few pieces of tensors
// ---------------------------------------------------------------------------------------------
//
// What a ragged tile takes is the chain of trips to memory in front of its last store: in a launch of a few tiles nothing
// else is under way, and in one of many such tiles a wavefront does nothing but wait.  The general path has five such trips
// and more (segment lengths, pointers, whole vectors; pointers and values of the single elements left over) and runs some 400
// instructions; a tile of one piece here has two, its pointers through the scalar unit and all of its data.  GPU time per
// launch, us, before and after (an empty launch takes 1.54): one tensor of 101 elements, 8 workers, binary32: pack 2.97 /
// 2.00, pipeline 2.90 / 2.05, unpack_update 2.43 / 1.61; 10 tiles and a ragged one, 3 workers: pipeline 3.59 / 2.26, 12 workers
// 6.47 / 2.99, 32 workers 13.0 / 5.8.  In the table form, 600 tensors of 301 elements, each a group: pipeline 3 workers 6.2 /
// 3.9, 8 workers 7.5 / 5.5, 16 workers 10.0 / 8.7; in groups of eight 7.2 / 5.6, 7.1 / 6.4, 9.4 / 8.4.

// Tile-local elements [lo, hi) are the elements from `off` on of tensor `layer`.
struct Piece {
    int layer, lo, hi;
    int64_t off;
    __device__ __forceinline__ int len() const { return hi - lo; }
    __device__ __forceinline__ int lanes() const { return (hi - lo + VEC - 1) / VEC; }
    // First element of the vector lane k takes.  The last one ends with the piece and so overlaps the one before it where
    // the piece is no whole number of vectors.  That is harmless in workgroups of one wavefront (HAVE_PIECES), which has read
    // all it needs of both before it writes, and both lanes write the same values; a second wavefront could read w and v after
    // the first has updated them.
    __device__ __forceinline__ int element(int k) const { return min(k * VEC, len() - VEC); }
};

// One piece by itself: its pointers are the same for all lanes.  Of a full tile, too, in the burst form.
template <int KIND, typename GradT, int PT, bool WVNT, int GENERAL = MGWFBP_GENERAL_GROUP>
__device__ __forceinline__ void one_piece(const CallArgs<GradT>& A, const WorkerPtrs<GradT, PT>& mrg, int64_t tile_base, const Piece& s,
                                          int lane) {
    static_assert(BLOCK == 64 || KIND < 0, "lanes that share elements are in one wavefront");
    WorkerPtrs<const GradT, PT> src;
    float* wp = nullptr;
    float* vp = nullptr;
    if constexpr (reads_grads(KIND)) src.fetch(A.grad_ptrs, A.L, s.layer, worker_base<KIND>());
    if constexpr (updates(KIND)) {
        wp = ro(A.w_ptrs)[s.layer];
        vp = ro(A.v_ptrs)[s.layer];
    }
    if (lane < s.lanes()) {
        const int e = s.element(lane);
        paced_step<KIND, GradT, PT, VEC, 1, WVNT, MGWFBP_TOGETHER, GENERAL>(A, src, mrg, wp, vp, s.off + e, tile_base + s.lo + e, 0);
    }
}

// Several pieces: each lane takes a vector of one of them and fetches that tensor's pointers itself; pieces shorter than a
// vector go element by element.  The vectors of a full tile are one too many for the lanes where two tensors meet inside a
// vector: then the pieces are taken as many at a time as there are lanes for (a piece never in two parts, see element()).
template <int KIND, typename GradT, int PT, typename Pieces>
__device__ __forceinline__ void several_pieces(const CallArgs<GradT>& A, const WorkerPtrs<GradT, PT>& mrg, int64_t tile_base, Pieces pieces) {
    static_assert(BLOCK == 64 || KIND < 0, "lanes that share elements are in one wavefront");
    int lane = static_cast<int>(threadIdx.x);
    here_only_per_lane(lane);
    Piece s;
    bool more = pieces.next(s);
    while (more) {
        int used = 0, layer = 0, at = 0;
        int64_t off = 0;
        for (; more && used + s.lanes() <= BLOCK; more = pieces.next(s)) {
            if (s.len() < VEC) {
                if (lane < s.len()) do_one<KIND, GradT, PT, 1>(A, mrg, s.layer, s.off + lane, tile_base + s.lo + lane);
                continue;
            }
            if (lane >= used) {                            // lanes past this piece get the next one's, or stay idle
                layer = s.layer;
                at = s.lo + s.element(lane - used);
                off = s.off + s.element(lane - used);
            }
            used += s.lanes();
        }
        if (lane < used) do_one<KIND, GradT, PT, VEC>(A, mrg, layer, off, tile_base + at);
    }
}

// ---------------------------------------------------------------------------------------------
// general path
// ---------------------------------------------------------------------------------------------

// Inclusive prefix sum across the lanes of the workgroup: shift-and-add inside each wavefront,
// wavefront totals combined through LDS.  Every lane of the workgroup must call it.
__device__ __forceinline__ int block_inclusive_scan(int tid, int x, int* s_wave) {
    const int lane = tid & 63;
    const int wave = tid >> 6;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    if (lane == 63) s_wave[wave] = x;
    __syncthreads();
    int carry = 0;
#pragma unroll
    for (int q = 0; q < BLOCK / 64; ++q)
        if (q < wave) carry += s_wave[q];
    return x + carry;
}

template <int KIND, typename GradT, int PT>
__device__ void general_tile(const Args<GradT>& A, const WorkerPtrs<GradT, PT>& mrg, const TileHdr& h,
                             int64_t tile_base, int clo, int chi, int* s_loc, int* s_layer, int* s_wave,
                             int* s_ragged, int* s_nragged) {
    // Only tile-local elements [clo, chi) are touched; 0 <= clo < chi <= h.valid.
    //
    // A lane takes the 4-element vectors it owns whole where it can.  A vector that is not wanted whole (it
    // crosses a tensor boundary, the end of the group or a clip edge) is set aside in LDS, and once every whole
    // vector is under way the elements of those vectors are dealt out one per lane: a tile pays for its ragged
    // spots with one more step, not with up to four dependent ones in a row on a single lane while the
    // rest of the workgroup waits.
    int tid = threadIdx.x;
    here_only_per_lane(tid);
    const SegTables seg = seg_tables(A);
    const int valid = h.valid;
    const int nseg = h.nseg;
    const int p_first = (clo & ~(VEC - 1)) + tid * VEC;
    const bool staged = needs_owner(KIND) && nseg <= MAXSEG;     // uniform over the workgroup
    __syncthreads();                            // the previous tile's readers are done with LDS
    if (tid == 0) *s_nragged = 0;
    if (staged) {
        // Tile-local start of segment j (1 <= j < nseg) = first_end + sum of the lengths of the
        // segments 1..j-1, all of which lie wholly inside the tile.  Each lane owns entries
        // j = 1 + 2*tid and j = 2 + 2*tid.
        const int j0 = 1 + 2 * tid, j1 = j0 + 1;
        int x0 = 0, x1 = 0;
        if (j0 < nseg) x0 = (j0 == 1) ? h.first_end : static_cast<int>(ro(seg.n)[h.seg0 + j0 - 1]);
        if (j1 < nseg) x1 = static_cast<int>(ro(seg.n)[h.seg0 + j1 - 1]);
        const int incl = block_inclusive_scan(tid, x0 + x1, s_wave);
        if (j0 < nseg) s_loc[j0] = incl - x1;
        if (j1 < nseg) s_loc[j1] = incl;
        for (int j = tid; j < nseg; j += BLOCK) s_layer[j] = ro(seg.layer)[h.seg0 + j];
        if (tid == 0) s_loc[nseg] = valid;
    }
    __syncthreads();
    auto start_of = [&](int j) -> int {         // j >= 1
        return staged ? s_loc[j] : static_cast<int>(static_cast<int64_t>(ro(seg.off)[h.seg0 + j]) - tile_base);
    };
    auto end_of = [&](int j) -> int { return (j + 1 < nseg) ? start_of(j + 1) : valid; };
    auto layer_of = [&](int j) -> int { return staged ? s_layer[j] : ro(seg.layer)[h.seg0 + j]; };
    auto owner_of = [&](int q) -> int {         // last j with start_of(j) <= q (segment 0 starts <= 0)
        int lo = 0, hi = nseg - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (start_of(mid) <= q) lo = mid; else hi = mid - 1;
        }
        return lo;
    };
    auto offset_in = [&](int j, int q) -> int64_t {   // element q of the tile is this element of segment j
        return (j == 0) ? (static_cast<int64_t>(q) - h.first_start) : static_cast<int64_t>(q - start_of(j));
    };
    for (int p = p_first; p < chi; p += BLOCK * VEC) {
        bool whole = p >= clo && p + VEC <= chi;
        int j = 0;
        if constexpr (needs_owner(KIND)) {
            j = owner_of(max(p, clo));
            whole = whole && p + VEC <= end_of(j);
        }
        if (whole) {
            if constexpr (needs_owner(KIND)) do_one<KIND, GradT, PT, VEC>(A, mrg, layer_of(j), offset_in(j, p), tile_base + p);
            else do_one<KIND, GradT, PT, VEC>(A, mrg, 0, 0, tile_base + p);
        } else {
            s_ragged[atomicAdd(s_nragged, 1)] = p;      // at most TILE / VEC entries: one per vector of the tile
        }
    }
    __syncthreads();
    const int n_ragged = *s_nragged;
    for (int e = tid; e < n_ragged * VEC; e += BLOCK) {
        const int q = s_ragged[e / VEC] + (e % VEC);
        if (q < clo || q >= chi) continue;
        if constexpr (needs_owner(KIND)) {
            const int j = owner_of(q);
            do_one<KIND, GradT, PT, 1>(A, mrg, layer_of(j), offset_in(j, q), tile_base + q);
        } else {
            do_one<KIND, GradT, PT, 1>(A, mrg, 0, 0, tile_base + q);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// the kernel
// ---------------------------------------------------------------------------------------------
typedef int i32x4 __attribute__((ext_vector_type(4)));

// The 32-byte tile header, fetched as two 16-byte read-only loads (wave-uniform address).
__device__ __forceinline__ TileHdr load_header(const TileHdr* p) {
    const MGWFBP_CONST i32x4* q = (const MGWFBP_CONST i32x4*)p;
    const i32x4 a = q[0], b = q[1];
    TileHdr h;
    h.first_start = static_cast<int64_t>((static_cast<uint64_t>(static_cast<uint32_t>(a[1])) << 32) |
                                         static_cast<uint32_t>(a[0]));
    h.first_end = a[2];
    h.seg0 = a[3];
    h.nseg = b[0];
    h.valid = b[1];
    h.layer0 = b[2];
    h.flags = b[3];
    return h;
}

// The pieces of a tile in the table form.
template <int KIND, typename GradT> struct TablePieces {
    const TileHdr& h;
    int clo, chi;
    SegTables seg;
    int j = 0, end = 0;
    __device__ __forceinline__ bool only(Piece& s) const {
        if constexpr (needs_owner(KIND)) {
            s = Piece{h.layer0, clo, chi, clo - h.first_start};
            return h.nseg == 1;
        } else {
            s = Piece{0, clo, chi, 0};
            return true;
        }
    }
    __device__ __forceinline__ bool next(Piece& s) {
        if constexpr (!needs_owner(KIND)) {
            s = Piece{0, clo, chi, 0};
            return j++ == 0;
        }
        if (j >= h.nseg) return false;
        int64_t start = h.first_start;
        s.layer = h.layer0;
        if (j == 0) {
            end = h.first_end;
        } else {
            start = end;
            s.layer = ro(seg.layer)[h.seg0 + j];
            end = j + 1 < h.nseg ? end + static_cast<int>(ro(seg.n)[h.seg0 + j]) : h.valid;
        }
        s.lo = j == 0 ? clo : max(static_cast<int>(start), clo);
        s.hi = min(end, chi);
        s.off = s.lo - start;
        ++j;
        return true;
    }
};

// FORM: vectors per lane a fast tile is walked in (1, see paced_step), BURST or PAIRS.
// 16-bit gradients run uncapped in single tiles and want the wavefronts; where the compiler stops a few registers short of one more,
// it is told the number per SIMD.  So it is in pairs of binary16 where the worker count is not compiled, which take 95 registers
// otherwise, 63 so (table form; 96 and 79 in the few-segments form).
template <int KIND, typename GradT, int PT, int FORM> constexpr int wanted_waves() {
    if (sizeof(GradT) != 2 || KIND != K_PIPELINE || PT != 0) return 1;
    return FORM == 1 ? 8 : FORM == PAIRS ? 6 : 1;
}

// Most pieces of a tile that are taken one after the other, see MGWFBP_PIECES.  Paced steps of 16-bit gradients that store
// nothing between the workers: the general path is ahead with 16 workers, and with 8 a reduce_update is left registers for 32
// wavefronts per compute unit instead of 28.  us with pieces / without, 300 tensors of log-normal sizes, bfloat16: direct, 16
// workers, 4700 tiles 15.5 / 14.4, reduce_update 11.8 / 11.5; a thousand around 1000 elements in groups of four 16.8 / 15.7; 8
// workers, 8000 tiles 13.7 / 12.4, 4700 tiles 8.5 / 8.6.  Fewer workers gain from pieces (direct, 4 workers, 4700 tiles 7.3 / 8.2), and so does
// a direct step of 16 where most tiles are ragged, which the launch says (thousands of tensors around 100 elements in groups of
// four, 9700 / 17,200 / 37,300 tiles 33.9 / 35.6, 54.5 / 58.4, 106.6 / 116.3; around 230 and 400 elements level).
template <int KIND, typename GradT, int PT, int FORM> constexpr int most_pieces() {
    constexpr bool one = FORM != BURST && sizeof(GradT) == 2 && ((directs(KIND) && PT == 16) || (reduce_updates(KIND) && (PT == 8 || PT == 16)));
    return one ? 1 : MGWFBP_PIECES;
}

template <int ROLE, typename GradT, int PT, int KERNEL_FORM>
__global__ void __launch_bounds__(MGWFBP_BLOCK, (wanted_waves<ROLE, GradT, PT, KERNEL_FORM>())) mgwfbp_stream_kernel(const Args<GradT> A) {
    constexpr int KIND = kind_in(ROLE, KERNEL_FORM);
    constexpr int FORM = single_steps(KERNEL_FORM) ? 1 : KERNEL_FORM;
    constexpr bool SHIFTS = KERNEL_FORM == ON_LINES;
    constexpr int SINGLE = FORM == PAIRS ? 1 : FORM;     // single tiles
    constexpr int JOIN = joined_tiles_of(KIND, FORM);
    constexpr int MOST = most_pieces<KIND, GradT, PT, FORM>();
    __shared__ int s_loc[MAXSEG + 1];
    __shared__ int s_layer[MAXSEG];
    __shared__ int s_wave[BLOCK / 64];
    __shared__ int s_ragged[TILE / VEC];
    __shared__ int s_nragged;
    __shared__ __align__(16) float s_sums[FORM == PAIRS ? PAIRED : 4];

    asm volatile("" ::"s"(A.tile_count), "s"(A.tile_first), "s"(static_cast<int>(A.tiles_per_wg)), "s"(A.tiles), "s"(A.n_units), "s"(A.turn),
                 "s"(static_cast<int>(A.clip_lo)), "s"(static_cast<int>(A.clip_hi)), "s"(A.merge_bufs), "s"(A.grad_ptrs), "s"(A.reduced),
                 "s"(A.inv_p), "s"(A.P));
    if constexpr (updates(KIND)) asm volatile("" ::"s"(A.w_ptrs), "s"(A.v_ptrs), "s"(A.lr));      // (see mgwfbp_few_kernel)

    WorkerPtrs<GradT, PT> mrg;
    if constexpr (reads_merge(KIND) || writes_merge(KIND)) mrg.fetch(A.merge_bufs, 1, 0, worker_base<KIND>());

    // Work is dealt in units of `tiles_per_wg` consecutive tiles.
    const int K = A.tiles_per_wg;
    const int n_units = A.n_units;              // ceil(tile_count / K), computed on the host
    int u_begin, u_end, u_step;
    if (A.flags & XCD_CONTIGUOUS) {
        // workgroup ids are dealt round-robin to the 8 dies: die = id % 8.  Give each die one
        // contiguous eighth of the units.
        const int die = blockIdx.x & 7;
        const int per_die = (n_units + 7) >> 3;
        u_begin = die * per_die + static_cast<int>(blockIdx.x >> 3);
        u_end = min(n_units, (die + 1) * per_die);
        u_step = A.turn >> 3;
    } else {
        u_begin = unit_of(A);
        u_end = n_units;
        u_step = A.turn;
    }
    for (int u = u_begin; u < u_end; u += u_step) {
        const int t_end = min((u + 1) * K, A.tile_count);
        for (int t = u * K; t < t_end; ++t) {
            int tile = A.tile_first + t;
            if constexpr (!directs(KIND)) here_only(tile);     // (addresses that run on from tile to tile would be set up, pointers waited for, first)
            const TileHdr h = load_header(A.tiles + tile);
            const int64_t tile_base = static_cast<int64_t>(tile) * TILE;
            const int clo = t == 0 ? A.clip_lo : 0;
            int chi = t == A.tile_count - 1 ? min(h.valid, static_cast<int>(A.clip_hi)) : h.valid;
            if (chi <= clo) continue;
            if constexpr (SHIFTS) {
                // The tile's share of a tensor begins on a line of the weights (see on_lines_pays()).  Whether the tensor goes on is in the
                // header, and the next tile's is read where it does only: reading both in front of every tile cost up to 7 % (100,000 tiles, 1
                // worker).  Launches are over whole groups, so a tensor that goes on does so in the launch's next tile.
                constexpr int LINE = line_elems(KIND, sizeof(GradT));
                auto shift_of = [&](const TileHdr& x) { return line_shift(reinterpret_cast<uint64_t>(ro(A.w_ptrs)[x.layer0]), x.first_start, LINE); };
                const bool goes_on = (h.flags & TILE_GOES_ON) != 0;
                int ahead = shift_of(h);
                if (h.nseg == 1 && goes_on && -h.first_start >= ahead) {
                    if (h.flags & TILE_RESIDENT) {             // (see below)
                        asm volatile("; w and v cacheable" ::: "memory");
                        fast_chunk<KIND, GradT, PT, NT_WV, 1>(A, mrg, h.layer0, -h.first_start - ahead, tile_base - ahead, TVECS);
                        asm volatile("; end w and v cacheable" ::: "memory");
                    } else {
                        asm volatile("; w and v streamed" ::: "memory");
                        fast_chunk<KIND, GradT, PT, true, 1>(A, mrg, h.layer0, -h.first_start - ahead, tile_base - ahead, TVECS);
                        asm volatile("; end w and v streamed" ::: "memory");
                    }
                    continue;
                }
                // A tile that a tensor begins or ends in: what lies before the tile, then the rest up to the next one's share.
                ahead = starts_early(h.first_start, ahead);
                int left = 0;
                if (goes_on) {
                    const TileHdr next = load_header(A.tiles + tile + 1);
                    left = starts_early(next.first_start, shift_of(next));
                }
                const Piece s{h.layer0, -ahead, 0, -h.first_start - ahead};
                int lane = threadIdx.x;
                here_only_per_lane(lane);
                if (ahead >= VEC) {
                    if (h.flags & TILE_RESIDENT) {
                        asm volatile("; w and v cacheable" ::: "memory");
                        one_piece<KIND, GradT, PT, NT_WV>(A, mrg, tile_base, s, lane);
                        asm volatile("; end w and v cacheable" ::: "memory");
                    } else {
                        asm volatile("; w and v streamed" ::: "memory");
                        one_piece<KIND, GradT, PT, true>(A, mrg, tile_base, s, lane);
                        asm volatile("; end w and v streamed" ::: "memory");
                    }
                } else if (lane < ahead) do_one<KIND, GradT, PT, 1>(A, mrg, s.layer, s.off + lane, tile_base + s.lo + lane);
                chi -= left;
            }
            const bool full = clo == 0 && chi == TILE && (!needs_owner(KIND) || h.nseg == 1);
            if constexpr (HAVE_PIECES) {
                TablePieces<KIND, GradT> pieces{h, clo, chi};
                Piece s;
                if ((FORM == BURST || !full) && pieces.only(s) && s.len() >= VEC) {
                    int lane = threadIdx.x;
                    here_only_per_lane(lane);
                    if (!updates(KIND) || (h.flags & TILE_RESIDENT)) {             // (see below)
                        asm volatile("; w and v cacheable" ::: "memory");
                        one_piece<KIND, GradT, PT, NT_WV>(A, mrg, tile_base, s, lane);
                        asm volatile("; end w and v cacheable" ::: "memory");
                    } else {
                        asm volatile("; w and v streamed" ::: "memory");
                        one_piece<KIND, GradT, PT, true>(A, mrg, tile_base, s, lane);
                        asm volatile("; end w and v streamed" ::: "memory");
                    }
                    continue;
                }
                if (!full && (!needs_owner(KIND) || h.nseg <= (directs(KIND) && MOST == 1 && (A.flags & IN_PIECES) ? MGWFBP_PIECES : MOST))) {
                    pieces.seg = seg_tables(A);
                    several_pieces<KIND, GradT, PT>(A, mrg, tile_base, pieces);
                    continue;
                }
            }
            if (!full) {
                general_tile<KIND, GradT, PT>(A, mrg, h, tile_base, clo, chi, s_loc, s_layer, s_wave, s_ragged, &s_nragged);
                continue;
            }
            if constexpr (HAVE_PIECES && FORM == BURST) continue;      // taken above
            // A full tile inside one tensor.
            if constexpr (JOIN > 1) {
                // (A clip cuts into the first and the last tile only.)
                if (t + JOIN <= t_end) {
                    bool same = t + JOIN < A.tile_count || A.clip_hi == TILE;
                    int flags = h.flags;
#pragma unroll
                    for (int k = 1; k < JOIN; ++k) {
                        const TileHdr hk = load_header(A.tiles + tile + k);
                        same = same && hk.valid == TILE && hk.nseg == 1 && hk.layer0 == h.layer0;
                        flags |= hk.flags;
                    }
                    if (same && (!updates(KIND) || !(flags & TILE_RESIDENT))) {
                        joined_tiles<KIND, GradT, PT>(A, mrg, h.layer0, -h.first_start, tile_base, s_sums);
                        t += JOIN - 1;
                        continue;
                    }
                }
            }
            // Tiles flagged "resident" keep their w and v in the memory-side cache between iterations
            // (ordinary loads and stores); all other w, v traffic is streamed past it like the gradients.
            // The two arms differ only in the cache policy of their memory instructions; the empty asm
            // statements keep the optimiser from merging them back into one (which drops the policy).
            const int64_t toff = -h.first_start;
            if constexpr (may_roll(KIND, FORM)) {
                if ((A.flags & ROLLING) && !(h.flags & TILE_RESIDENT)) {
                    rolling_tile<GradT, PT>(A, mrg, h.layer0, toff, tile_base);
                    continue;
                }
            }
            if (!updates(KIND) || (h.flags & TILE_RESIDENT)) {
                asm volatile("; w and v cacheable" ::: "memory");
                fast_chunk<KIND, GradT, PT, NT_WV, SINGLE>(A, mrg, h.layer0, toff, tile_base, TVECS);
                asm volatile("; end w and v cacheable" ::: "memory");
            } else {
                asm volatile("; w and v streamed" ::: "memory");
                fast_chunk<KIND, GradT, PT, true, SINGLE>(A, mrg, h.layer0, toff, tile_base, TVECS);
                asm volatile("; end w and v streamed" ::: "memory");
            }
        }
    }
}

// ---------------------------------------------------------------------------------------------
// the same for a launch over at most FEW segments, which come along as arguments
// ---------------------------------------------------------------------------------------------
//
// One group, or a tensor that has just arrived, is a handful of segments, and a launch over it is short enough
// that the trips to memory in front of the first gradient count: the tile header, then the segment lengths of a
// ragged tile, their prefix sum through LDS, and the search in it.  Here a workgroup works all of that out from
// its arguments in scalar registers, so only the pointers lie between it and its data.  Segment j is tensor
// layer_hi - j and starts where j - 1 ends, or on the next tile after the last segment of a group.  Kinds that
// need no tensors (REDUCE) get whole groups as segments.
template <typename GradT> __device__ __forceinline__ int few_start(const FewArgs<GradT>& A, int j) {   // j static
    if (j == 0) return A.start0;
    const int e = A.end[j - 1];
    return (A.closes >> (j - 1)) & 1 ? (e + TILE - 1) & ~(TILE - 1) : e;
}

// Segment that element q belongs to if it belongs to any: the last one that starts at or before q, or segment 0.  (Past the
// segments there are lie empty ones; who they own does not matter.)
struct FewSeg { int j, start, end; };
template <typename GradT> __device__ __forceinline__ FewSeg few_owner(const FewArgs<GradT>& A, int q) {
    FewSeg s{0, A.start0, A.end[0]};
#pragma unroll
    for (int j = 1; j < FEW; ++j) {
        const int start = few_start(A, j);
        if (q >= start) s = FewSeg{j, start, A.end[j]};
    }
    return s;
}

// Whether the ends of all segments come with the other arguments.  Where they do, a tile that needs them has them a trip
// earlier; where they do not, the single tensors of long launches have the scalar registers.  us with the ends in the general
// part only / with the other arguments, burst form: three tensors of 300 elements, 8 workers, binary32: pipeline 2.63 / 2.40,
// reduce_update 2.55 / 2.36; seven of 9 to 2000, 16 workers, bfloat16: 4.05 / 3.55, 3.37 / 3.02; pack 2.56 / 2.25.
constexpr bool ends_early(int kind, int form) { return form == BURST || kind == K_PACK; }

// One tile of the few-segments form (of PACK or in pairs: a joined step); the tiles taken.
template <int KIND, typename GradT, int PT, int FORM>
__device__ __forceinline__ int few_tile(const FewArgs<GradT>& A, const MGWFBP_CONST FewArgs<GradT>* a, int t, int t_end, float* s_sums) {
    constexpr int SINGLE = FORM == PAIRS ? 1 : FORM;
    constexpr int JOIN = joined_tiles_of(KIND, FORM);
    constexpr bool EARLY = ends_early(KIND, FORM);
    // Paced steps of 16-bit gradients that store nothing between 16 workers want every wave slot (see few_form_pays): their
    // ragged tiles go in groups of eight.
    constexpr bool TIGHT = PT == 16 && sizeof(GradT) == 2 && FORM == 1 && !writes_merge(KIND);
    constexpr int LANES = TIGHT ? 0 : PT;
    const int64_t arena = static_cast<int64_t>(A.tile_first) * TILE;
    const int b = t * TILE;
    auto mrg = [&](auto count) {                                       // (fetched where it is used: 16 workers have no registers to keep it in)
        WorkerPtrs<GradT, decltype(count)::value> m;
        if constexpr (reads_merge(KIND) || writes_merge(KIND)) m.fetch(A.merge_bufs, 1, 0, worker_base<KIND>());
        return m;
    };
    // Segment that ends in the tile or beyond it (the last one does); all of the tile's if it is the last one or ends
    // beyond it.
    int j = 0, start = A.start0, end = A.end[0];
    auto next = [&](int i, int its_end) {
        start = (A.closes >> i) & 1 ? (end + TILE - 1) & ~(TILE - 1) : end;
        end = its_end;
        j = i + 1;
    };
    if constexpr (EARLY) {
#pragma unroll
        for (int i = 0; i < FEW - 1; ++i) {
            if (end > b) break;
            next(i, A.end[i + 1]);
        }
    } else {
        while (end <= b && j < FEW - 1) next(j, a->end[j + 1]);        // read where they lie: the index need not be known beforehand
    }
    if (FORM != BURST && start <= b && b + TILE <= end) {              // a full tile inside one segment
        if constexpr (JOIN > 1) {
            if (t + JOIN <= t_end && b + JOIN * TILE <= end) {
                joined_tiles<KIND, GradT, PT>(A, mrg(Int<PT>()), A.layer_hi - j, b - start, arena + b, s_sums);
                return JOIN;
            }
        }
        if constexpr (may_roll(KIND, FORM)) {
            if (A.flags & ROLLING) {
                asm volatile("; rolling steps" ::: "memory");      // keeps the arms' addresses, and their registers, apart
                rolling_tile<GradT, PT>(A, mrg(Int<PT>()), A.layer_hi - j, b - start, arena + b);
                asm volatile("; end rolling steps" ::: "memory");
                return 1;
            }
            asm volatile("; single steps" ::: "memory");
        }
        fast_chunk<KIND, GradT, PT, true, SINGLE>(A, mrg(Int<PT>()), A.layer_hi - j, b - start, arena + b, TVECS);
        return 1;
    }
    const Piece s{A.layer_hi - j, max(start - b, 0), min(end - b, TILE), b + max(start - b, 0) - start};
    const bool only = j + 1 >= A.n || end >= b + TILE || ((A.closes >> j) & 1);
    if (only && s.len() >= VEC) {
        one_piece<KIND, GradT, PT, true, TIGHT ? 8 : MGWFBP_GENERAL_GROUP>(A, mrg(Int<PT>()), arena + b, s, threadIdx.x);
        return 1;
    }
    // Whole vectors first, then the wanted elements of the others, one per lane (see general_tile).  (Where segments start is
    // worked out here only, see here_only.)
    FewArgs<GradT> B = A;
    if constexpr (EARLY) {
        int32_t closes = A.closes;
        here_only(closes);
        B.closes = static_cast<uint8_t>(closes);
    } else {
        asm volatile("" : "+s"(a));
        B = *(const FewArgs<GradT>*)a;
    }
    int lane = threadIdx.x;
    here_only_per_lane(lane);
    const int p = b + lane * VEC;
    const FewSeg o = few_owner(B, p);
    const bool whole = p >= o.start && p + VEC <= o.end;
    const bool any = (p < o.end && p + VEC > o.start) || few_owner(B, p + VEC - 1).j != o.j;
    const uint64_t ragged = __ballot(any && !whole);
    if (whole) do_one<KIND, GradT, LANES, VEC>(A, mrg(Int<LANES>()), A.layer_hi - o.j, p - o.start, arena + p);
    const int n_ragged = __popcll(ragged) * VEC;
    for (int e = lane; e < n_ragged; e += BLOCK) {
        uint64_t rest = ragged;
        for (int k = e / VEC; k > 0; --k) rest &= rest - 1;
        const int q = b + __builtin_ctzll(rest) * VEC + e % VEC;
        const FewSeg r = few_owner(B, q);
        if (q >= r.start && q < r.end) do_one<KIND, GradT, LANES, 1>(A, mrg(Int<LANES>()), A.layer_hi - r.j, q - r.start, arena + q);
    }
    return 1;
}

// Wavefronts per SIMD that the compiler is told to leave registers for: 16 workers' loads take 98 registers in the burst form of
// a binary32 reduce_update otherwise (20 instead of 16 wavefronts per compute unit).
template <int KIND, typename GradT, int PT, int FORM> constexpr int wanted_few_waves() {
    if (FORM == PAIRS) return wanted_waves<KIND, GradT, PT, FORM>();
    return PT == 16 && KIND == K_REDUCE_UPDATE && sizeof(GradT) == 4 ? 5 : 1;
}

// Scalar registers bound the wavefronts of these kernels: a SIMD has 800, and a wavefront takes what it needs in blocks of 16
// and 16 more, so eight fit with up to 80, seven with up to 96 and six beyond (the compiler's own figure leaves the 16 out; seen
// where a launch no longer fits at once: 93 registers at 28 tiles per compute unit, 80 at 32, 103 at 24).  us with 83 to 103 / 55
// to 80, bfloat16, one tensor of 7500 tiles: direct, 4 / 8 / 16 / 32 workers 9.3 / 8.2, 12.7 / 10.6, 18.9 / 15.4, 29.9 / 24.9; reduce_update 9.3 / 8.3,
// 12.4 / 10.4, 18.1 / 15.2, 29.2 / 23.9.
template <int ROLE, typename GradT, int PT, int KERNEL_FORM>
__global__ void __launch_bounds__(MGWFBP_BLOCK, (wanted_few_waves<ROLE, GradT, PT, KERNEL_FORM>())) mgwfbp_few_kernel(FewArgs<GradT> A) {
    constexpr int KIND = kind_in(ROLE, KERNEL_FORM);
    constexpr int FORM = single_steps(KERNEL_FORM) ? 1 : KERNEL_FORM;
    static_assert(KIND >= 0 && HAVE_FEW, "a tile is one vector per lane of one wavefront");
    __shared__ __align__(16) float s_sums[FORM == PAIRS ? PAIRED : 4];
    // All arguments in one trip; left alone, the compiler fetches them where it needs them, in three.
    asm volatile("" ::"s"(A.tile_count), "s"(A.layer_hi), "s"(static_cast<int>(A.n)), "s"(A.end[0]), "s"(A.merge_bufs), "s"(A.grad_ptrs),
                 "s"(A.reduced), "s"(A.inv_p), "s"(A.P));
    if constexpr (updates(KIND)) asm volatile("" ::"s"(A.w_ptrs), "s"(A.v_ptrs), "s"(A.lr));
    if constexpr (ends_early(KIND, FORM))
        asm volatile("" ::"s"(A.end[1]), "s"(A.end[2]), "s"(A.end[3]), "s"(A.end[4]), "s"(A.end[5]), "s"(A.end[6]), "s"(A.end[7]));
    const MGWFBP_CONST FewArgs<GradT>* a = (const MGWFBP_CONST FewArgs<GradT>*)__builtin_amdgcn_kernarg_segment_ptr();
    int t = unit_of(A) * A.tiles_per_wg;
    const int t_end = min(t + A.tiles_per_wg, A.tile_count);
    while (t < t_end) {
        t += few_tile<KIND, GradT, PT, FORM>(A, a, t, t_end, s_sums);
        if (t >= t_end) break;
        // A further tile, where the caller asked for several: the arguments again, so that no path keeps them, or what the
        // compiler works out from them beforehand, in registers for it (10 scalar registers).  PACK takes several by itself and
        // has the registers (bfloat16, 32 workers, 40,000 tiles 198 us, with the arguments again 212).
        if constexpr (KIND != K_PACK) {
            asm volatile("" : "+s"(a));
            A = *(const FewArgs<GradT>*)a;
        }
    }
}

thread_local int g_last_hip_error = 0;

int note(hipError_t e) {
    if (e == hipSuccess) return MGWFBP_OK;
    g_last_hip_error = static_cast<int>(e);
    return MGWFBP_EHIP;
}

}  // namespace

int mgwfbp_note_hip_result(int hip_error_code) { return note(static_cast<hipError_t>(hip_error_code)); }

// ---------------------------------------------------------------------------------------------
// context
// ---------------------------------------------------------------------------------------------

struct mgwfbp_ctx {
    HostTables host;
    int32_t P = 0;
    int32_t dtype = 0;
    bool on_device = false;
    int device = -1;
    int n_cu = 0;
    LaunchSettings set;
    int32_t resident_end = 0;         // tiles up to here are resident, but for a few that did not fit
    uint64_t serial = 0;              // changes whenever the tables change; never reused within a process
    // device copies
    unsigned char* d_tables = nullptr;   // the segment tables and the tile headers, one block
    TileHdr* d_tiles = nullptr;          // the tile headers in it
};

namespace {

std::atomic<uint64_t> g_next_serial{1};

// Marks the leading tiles whose w + v bytes (8 per element) fit into the budget; the end of the last one marked.
int32_t mark_resident_tiles(HostTables& h, uint64_t budget) {
    uint64_t used = 0;
    int32_t end = 0;
    for (size_t i = 0; i < h.tiles.size(); ++i) {
        const uint64_t need = static_cast<uint64_t>(h.tiles[i].valid) * 8u;
        if (used + need <= budget) {
            h.tiles[i].flags |= TILE_RESIDENT;
            used += need;
            end = static_cast<int32_t>(i + 1);
        } else {
            h.tiles[i].flags &= ~TILE_RESIDENT;
        }
    }
    return end;
}

// Both parts of the block start on multiples of 256 bytes.
int upload_tables(mgwfbp_ctx* c) {
    const std::vector<unsigned char>& segs = c->host.seg_block;
    const size_t b_tiles = c->host.tiles.size() * sizeof(TileHdr);
    hipError_t e = hipMalloc(reinterpret_cast<void**>(&c->d_tables), segs.size() + b_tiles);
    if (e != hipSuccess) {
        c->d_tables = nullptr;
        g_last_hip_error = static_cast<int>(e);
        return e == hipErrorOutOfMemory ? MGWFBP_ENOMEM : MGWFBP_EHIP;
    }
    c->d_tiles = reinterpret_cast<TileHdr*>(c->d_tables + segs.size());
    int rc = note(hipMemcpy(c->d_tables, segs.data(), segs.size(), hipMemcpyHostToDevice));
    if (rc == MGWFBP_OK && b_tiles > 0) rc = note(hipMemcpy(c->d_tiles, c->host.tiles.data(), b_tiles, hipMemcpyHostToDevice));
    return rc;
}

int create_common(mgwfbp_ctx** out, const uint64_t* n_elems, int32_t L, const uint8_t* merged, int32_t P,
                  int32_t dtype, bool device) {
    if (out == nullptr) return MGWFBP_EINVAL;
    *out = nullptr;
    if (P < 1 || P > MGWFBP_MAX_P) return MGWFBP_EINVAL;
    if (dtype != MGWFBP_F32 && dtype != MGWFBP_BF16 && dtype != MGWFBP_F16) return MGWFBP_EINVAL;
    mgwfbp_ctx* c = new (std::nothrow) mgwfbp_ctx();
    if (c == nullptr) return MGWFBP_ENOMEM;
    int rc = mgwfbp_build_tables(n_elems, L, merged, c->host);
    if (rc != MGWFBP_OK) {
        delete c;
        return rc;
    }
    c->P = P;
    c->dtype = dtype;
    c->serial = g_next_serial.fetch_add(1);
    c->resident_end = mark_resident_tiles(c->host, c->set.resident_bytes);
    if (device) {
        hipDeviceProp_t prop;
        rc = note(hipGetDevice(&c->device));
        if (rc == MGWFBP_OK) rc = note(hipGetDeviceProperties(&prop, c->device));
        if (rc == MGWFBP_OK) {
            c->n_cu = prop.multiProcessorCount;
            rc = upload_tables(c);
        }
        if (rc != MGWFBP_OK) {
            mgwfbp_ctx_destroy(c);
            return rc;
        }
        c->on_device = true;
    }
    *out = c;
    return MGWFBP_OK;
}

// The launch itself, by the runtime's function and not by the <<<>>> syntax: that one leaves grid, LDS and stream with the
// runtime, calls a stub that fetches them again, and reports through hipGetLastError.
template <int KIND, typename GradT, int PT, int FORM, template <typename> class ArgsT>
int start(const ArgsT<GradT>& A, hipStream_t stream, const LaunchShape& s, int grid_y) {
    constexpr bool FEW_FORM = std::is_same<ArgsT<GradT>, FewArgs<GradT>>::value;
    const void* kernel;
    if constexpr (FEW_FORM) kernel = reinterpret_cast<const void*>(&mgwfbp_few_kernel<KIND, GradT, PT, FORM>);
    else kernel = reinterpret_cast<const void*>(&mgwfbp_stream_kernel<KIND, GradT, PT, FORM>);
    const size_t lds = lds_for_workgroups_per_cu(s.wgs_per_cu, static_lds(KIND, FEW_FORM, FORM));
    void* args[1] = {const_cast<ArgsT<GradT>*>(&A)};
    const hipError_t e = hipLaunchKernel(kernel, dim3(s.grid, grid_y), dim3(BLOCK), args, lds, stream);
    if (e != hipSuccess) (void)hipGetLastError();        // reported here, not to whoever asks next
    return note(e);
}

template <int KIND, typename GradT, int PT, template <typename> class ArgsT>
int launch_one(const ArgsT<GradT>& A, hipStream_t stream, const LaunchShape& s, int grid_y = 1) {
    if constexpr (KIND != K_PACK) {                       // PACK has one form
        if (s.form == BURST) return start<KIND, GradT, PT, BURST>(A, stream, s, grid_y);
    }
    constexpr bool TABLE = !std::is_same<ArgsT<GradT>, FewArgs<GradT>>::value;
    if constexpr (HAVE_PIECES && (KIND == K_UPDATE || KIND == K_DIRECT) && TABLE) {
        if (s.on_lines) return start<KIND, GradT, PT, ON_LINES>(A, stream, s, grid_y);
    }
    if constexpr (TVECS == 1 && TABLE && sizeof(GradT) == 4 && (KIND == K_REDUCE_UPDATE || KIND == K_DIRECT || KIND == K_PIPELINE)) {
        if (s.through) return start<KIND, GradT, PT, THROUGH>(A, stream, s, grid_y);
    }
    if constexpr (TVECS % 2 == 0) {
        if (s.form == 2) return start<KIND, GradT, PT, 2>(A, stream, s, grid_y);
    }
    if constexpr (HAVE_PAIRS && KIND == K_PIPELINE && sizeof(GradT) == 2) {
        if (s.form == PAIRS) return start<KIND, GradT, PT, PAIRS>(A, stream, s, grid_y);
    }
    return start<KIND, GradT, PT, 1>(A, stream, s, grid_y);
}

template <int KIND, typename GradT, template <typename> class ArgsT>
int launch_by_p(const ArgsT<GradT>& A, hipStream_t stream, const LaunchShape& s) {
    if constexpr (KIND == K_UPDATE) {
        return launch_one<KIND, GradT, 0>(A, stream, s);   // no per-worker data
    } else if constexpr (KIND == K_PACK) {
        return launch_one<KIND, GradT, 1>(A, stream, s, A.P);   // P independent single-worker copies
    } else {
        switch (A.P) {
            case 2: return launch_one<KIND, GradT, 2>(A, stream, s);
            case 4: return launch_one<KIND, GradT, 4>(A, stream, s);
            case 8: return launch_one<KIND, GradT, 8>(A, stream, s);
            case 16: return launch_one<KIND, GradT, 16>(A, stream, s);
            default: return launch_one<KIND, GradT, 0>(A, stream, s);
        }
    }
}

// Tile range and element clip of one call: either a group (or all groups), or an arena interval.
struct Span {
    int32_t t0 = 0, t1 = 0;               // tiles
    int32_t s0 = 0, s1 = 0;               // segments
    int32_t g0 = 0, g1 = 0;               // groups (not set for a clipped span)
    bool clipped = false;
    int64_t lo = 0, hi = 0;
};

Span span_of_groups(const HostTables& h, int32_t g0, int32_t g1) {
    Span s;
    s.t0 = h.group_tile[static_cast<size_t>(g0)];
    s.t1 = h.group_tile[static_cast<size_t>(g1)];
    s.s0 = h.group_seg[static_cast<size_t>(g0)];
    s.s1 = h.group_seg[static_cast<size_t>(g1)];
    s.g0 = g0;
    s.g1 = g1;
    return s;
}

// Fills in the segments of a launch if it can take the few-segments form: at most FEW of them, of consecutive
// tensors (no empty tensor in between), less than 2^30 elements in all.
bool few_segments(const HostTables& h, const Span& sp, bool whole_groups, int32_t& layer_hi, int16_t& start0, uint8_t& n_out,
                  uint8_t& closes, int32_t* end) {
    const int64_t base = static_cast<int64_t>(sp.t0) * TILE;
    if (static_cast<int64_t>(sp.t1 - sp.t0) * TILE > (1 << 30)) return false;
    int n = 0;
    layer_hi = 0;
    start0 = 0;
    closes = 0;
    if (whole_groups) {                                // REDUCE: a segment is all of a group
        if (sp.g1 - sp.g0 > FEW) return false;
        for (int32_t k = sp.g0; k < sp.g1; ++k) {
            const size_t q = static_cast<size_t>(k);
            if (h.group_elems[q] == 0) continue;
            closes = static_cast<uint8_t>(closes | 1u << n);
            end[n++] = static_cast<int32_t>(static_cast<int64_t>(h.group_base[q] + h.group_elems[q]) - base);
        }
    } else {
        if (sp.s1 - sp.s0 > FEW) return false;
        const size_t s0 = static_cast<size_t>(sp.s0);
        layer_hi = h.seg_layer[s0];
        start0 = static_cast<int16_t>(static_cast<int64_t>(h.seg_off[s0]) - base);
        for (; n < sp.s1 - sp.s0; ++n) {
            const size_t q = static_cast<size_t>(layer_hi - n);
            if (h.seg_layer[s0 + static_cast<size_t>(n)] != layer_hi - n) return false;
            if (n + 1 < sp.s1 - sp.s0 && h.tensor_group[q] != h.tensor_group[q - 1])
                closes = static_cast<uint8_t>(closes | 1u << n);
            end[n] = static_cast<int32_t>(static_cast<int64_t>(h.seg_off[s0 + static_cast<size_t>(n)] + h.tensor_n[q]) - base);
        }
    }
    n_out = static_cast<uint8_t>(n);
    for (int j = n; j < FEW; ++j) end[j] = end[n - 1];
    return n > 0;
}

// Fills the argument block of the form the launch takes, and launches.
template <int KIND, typename GradT>
int launch(const mgwfbp_ctx* c, const Span& sp, const TileHdr* tiles, const CallArgs<GradT>& call,
           hipStream_t stream, const LaunchShape& s) {
    if constexpr (HAVE_FEW) {
        FewArgs<GradT> A{call};
        if (s.may_be_few && few_segments(c->host, sp, !needs_owner(KIND), A.layer_hi, A.start0, A.n, A.closes, A.end))
            return launch_by_p<KIND, GradT, FewArgs>(A, stream, s);
    }
    // a clip cuts into the first and the last tile only
    const int16_t clip_lo = static_cast<int16_t>(sp.clipped ? sp.lo - static_cast<int64_t>(sp.t0) * TILE : 0);
    const int16_t clip_hi = static_cast<int16_t>(sp.clipped ? sp.hi - static_cast<int64_t>(sp.t1 - 1) * TILE : TILE);
    const Args<GradT> A{call, tiles, static_cast<int32_t>(c->host.seg_layer.size()), s.units, s.grid, clip_lo, clip_hi};
    return launch_by_p<KIND, GradT, Args>(A, stream, s);
}

template <int KIND>
int run(mgwfbp_ctx* c, int32_t group, const void* const* grad_ptrs, void* const* merge_bufs, float* reduced,
        float* const* w_ptrs, float* const* v_ptrs, float lr, float mu, void* stream_v,
        const Span* span = nullptr, const TileHdr* static_tiles = nullptr) {
    if (c == nullptr || (static_tiles == nullptr && !c->on_device)) return MGWFBP_EINVAL;
    if (span == nullptr && (group < -1 || group >= c->host.G)) return MGWFBP_EINVAL;
    if (reads_grads(KIND) && grad_ptrs == nullptr) return MGWFBP_EINVAL;
    if ((reads_merge(KIND) || writes_merge(KIND)) && merge_bufs == nullptr) return MGWFBP_EINVAL;
    if ((KIND == K_REDUCE || KIND == K_UPDATE) && reduced == nullptr) return MGWFBP_EINVAL;
    if (updates(KIND) && (w_ptrs == nullptr || v_ptrs == nullptr)) return MGWFBP_EINVAL;

    Span sp;
    if (span != nullptr) sp = *span;
    else if (group < 0) sp = span_of_groups(c->host, 0, c->host.G);
    else sp = span_of_groups(c->host, group, group + 1);
    const int32_t count = sp.t1 - sp.t0;
    if (count <= 0) return MGWFBP_OK;             // nothing to move (empty group or empty model)

    // where the kernels find the tables: normally the context's own device copies
    const TileHdr* tiles = c->d_tiles;
    if (static_tiles != nullptr) {
        tiles = static_tiles;                         // the caller vouches for the current device
    } else {
        int dev = -1;
        int rc = note(hipGetDevice(&dev));
        if (rc != MGWFBP_OK) return rc;
        if (dev != c->device) return MGWFBP_EINVAL;   // tables live on the device the context was made on
    }

    const double resident = static_cast<double>(std::min(std::max(c->resident_end - sp.t0, 0), count)) / count;
    const LaunchShares shares = shares_of(c->host, sp.s0, sp.s1, count);
    const LaunchWork work{KIND, c->dtype, c->P, count, shares.ragged, shares.off_lines, reduced != nullptr, resident, sp.s1 - sp.s0};
    const LaunchShape s = launch_shape(c->set, work, c->n_cu);
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    const float inv_p = 1.0f / static_cast<float>(c->P);
    auto go = [&](auto grad) {
        typedef decltype(grad) GradT;
        const CallArgs<GradT> call{reinterpret_cast<const GradT* const*>(grad_ptrs), reinterpret_cast<GradT* const*>(merge_bufs),
                                   reduced, w_ptrs, v_ptrs, lr, mu, inv_p, c->host.L, c->P, sp.t0, count,
                                   static_cast<int16_t>(s.tiles_per_wg),
                                   static_cast<int8_t>((s.xcd_contiguous ? XCD_CONTIGUOUS : 0) | (s.rolling ? ROLLING : 0) | (s.in_pieces ? IN_PIECES : 0)), s.run_log2};
        return launch<KIND, GradT>(c, sp, tiles, call, stream, s);
    };
    if (c->dtype == MGWFBP_F32) return go(float{});
    if (c->dtype == MGWFBP_F16) return go(_Float16{});
    return go(uint16_t{});
}

// Per device: where that GPU's copy of `scratch` lives and whose tables it holds.
struct StaticSlot {
    unsigned char* ptr = nullptr;
    bool loaded = false;
    uint64_t serial = 0;              // context serial of the tables last written there
    hipStream_t stream = nullptr;     // ... and the stream the copy was ordered on
};
constexpr int MAX_STATIC_DEVICES = 64;
StaticSlot g_static[MAX_STATIC_DEVICES];
std::mutex g_static_mutex;

}  // namespace

extern "C" {

int mgwfbp_ctx_create(mgwfbp_ctx** ctx_out, const uint64_t* n_elems, int32_t L, const uint8_t* merged,
                      int32_t P, int32_t grad_dtype) {
    return create_common(ctx_out, n_elems, L, merged, P, grad_dtype, true);
}

int mgwfbp_ctx_create_host(mgwfbp_ctx** ctx_out, const uint64_t* n_elems, int32_t L, const uint8_t* merged,
                           int32_t P, int32_t grad_dtype) {
    return create_common(ctx_out, n_elems, L, merged, P, grad_dtype, false);
}

void mgwfbp_ctx_destroy(mgwfbp_ctx* c) {
    if (c == nullptr) return;
    if (c->d_tables) (void)hipFree(c->d_tables);
    delete c;
}

int mgwfbp_ctx_dims(const mgwfbp_ctx* c, int32_t* L, int32_t* n_groups, int32_t* P, int32_t* grad_dtype,
                    uint64_t* arena_elems, int32_t* tile_elems, int32_t* n_tiles) {
    if (c == nullptr) return MGWFBP_EINVAL;
    if (L) *L = c->host.L;
    if (n_groups) *n_groups = c->host.G;
    if (P) *P = c->P;
    if (grad_dtype) *grad_dtype = c->dtype;
    if (arena_elems) *arena_elems = c->host.arena_elems;
    if (tile_elems) *tile_elems = TILE;
    if (n_tiles) *n_tiles = static_cast<int32_t>(c->host.tiles.size());
    return MGWFBP_OK;
}

int mgwfbp_ctx_layout(const mgwfbp_ctx* c, uint64_t* tensor_off, int32_t* tensor_group, uint64_t* group_base,
                      uint64_t* group_elems) {
    if (c == nullptr) return MGWFBP_EINVAL;
    const HostTables& h = c->host;
    if (tensor_off && h.L) std::memcpy(tensor_off, h.tensor_off.data(), sizeof(uint64_t) * static_cast<size_t>(h.L));
    if (tensor_group && h.L) std::memcpy(tensor_group, h.tensor_group.data(), sizeof(int32_t) * static_cast<size_t>(h.L));
    if (group_base && h.G) std::memcpy(group_base, h.group_base.data(), sizeof(uint64_t) * static_cast<size_t>(h.G));
    if (group_elems && h.G) std::memcpy(group_elems, h.group_elems.data(), sizeof(uint64_t) * static_cast<size_t>(h.G));
    return MGWFBP_OK;
}

int mgwfbp_ctx_tables(const mgwfbp_ctx* c, int32_t* n_segments, void* tiles_out, uint64_t* seg_off_out,
                      uint32_t* seg_n_out, int32_t* seg_layer_out, int32_t* group_tile_out) {
    if (c == nullptr) return MGWFBP_EINVAL;
    const HostTables& h = c->host;
    const size_t S = h.seg_layer.size();
    if (n_segments) *n_segments = static_cast<int32_t>(S);
    if (tiles_out && !h.tiles.empty()) {
        std::memcpy(tiles_out, h.tiles.data(), sizeof(TileHdr) * h.tiles.size());
        for (size_t i = 0; i < h.tiles.size(); ++i) {
            const int32_t shown = h.tiles[i].flags & TILE_RESIDENT;
            std::memcpy(static_cast<unsigned char*>(tiles_out) + i * sizeof(TileHdr) + offsetof(TileHdr, flags), &shown, sizeof shown);
        }
    }
    if (seg_off_out) std::memcpy(seg_off_out, h.seg_off.data(), sizeof(uint64_t) * (S + 1));
    if (seg_n_out && S) std::memcpy(seg_n_out, h.seg_n.data(), sizeof(uint32_t) * S);
    if (seg_layer_out && S) std::memcpy(seg_layer_out, h.seg_layer.data(), sizeof(int32_t) * S);
    if (group_tile_out) std::memcpy(group_tile_out, h.group_tile.data(), sizeof(int32_t) * h.group_tile.size());
    return MGWFBP_OK;
}

int mgwfbp_ctx_set_launch(mgwfbp_ctx* c, int32_t blocks_per_cu, int32_t xcd_contiguous, int32_t tiles_per_workgroup) {
    if (c == nullptr || blocks_per_cu > 4096 || tiles_per_workgroup > 1024) return MGWFBP_EINVAL;
    c->set.tiles_per_wg = tiles_per_workgroup <= 0 ? 0 : tiles_per_workgroup;
    c->set.blocks_per_cu = blocks_per_cu <= 0 ? LaunchSettings{}.blocks_per_cu : blocks_per_cu;
    c->set.xcd_contiguous = xcd_contiguous ? 1 : 0;
    return MGWFBP_OK;
}

int mgwfbp_ctx_set_pacing(mgwfbp_ctx* c, int32_t workgroups_per_cu, int32_t vectors_per_step) {
    if (c == nullptr || workgroups_per_cu > 64 || vectors_per_step < -1 || vectors_per_step > TVECS ||
        (vectors_per_step > 0 && TVECS % vectors_per_step != 0))
        return MGWFBP_EINVAL;
    c->set.wg_per_cu = workgroups_per_cu;
    c->set.step_vecs = vectors_per_step;
    return MGWFBP_OK;
}

int mgwfbp_ctx_set_small_launch(mgwfbp_ctx* c, int32_t max_tiles) {
    if (c == nullptr) return MGWFBP_EINVAL;
    c->set.burst_tiles = max_tiles;
    return MGWFBP_OK;
}

int mgwfbp_ctx_set_resident_bytes(mgwfbp_ctx* c, uint64_t bytes) {
    if (c == nullptr) return MGWFBP_EINVAL;
    c->set.resident_bytes = bytes;
    c->serial = g_next_serial.fetch_add(1);
    c->resident_end = mark_resident_tiles(c->host, bytes);
    if (c->on_device && !c->host.tiles.empty())
        return note(hipMemcpy(c->d_tiles, c->host.tiles.data(), c->host.tiles.size() * sizeof(TileHdr),
                              hipMemcpyHostToDevice));
    return MGWFBP_OK;
}

int mgwfbp_pack(mgwfbp_ctx* c, int32_t group, const void* const* d_grad_ptrs, void* const* d_merge_bufs,
                void* hip_stream) {
    return run<K_PACK>(c, group, d_grad_ptrs, d_merge_bufs, nullptr, nullptr, nullptr, 0.f, 0.f, hip_stream);
}

int mgwfbp_pack_tensors(mgwfbp_ctx* c, int32_t first_tensor, int32_t last_tensor, const void* const* d_grad_ptrs,
                        void* const* d_merge_bufs, void* hip_stream) {
    if (c == nullptr || !c->on_device) return MGWFBP_EINVAL;
    const HostTables& h = c->host;
    if (last_tensor < 0 || first_tensor >= h.L || first_tensor < last_tensor) return MGWFBP_EINVAL;
    // Tensors lie in the arena in arrival order, so the run first_tensor, ..., last_tensor is a run of segments and
    // occupies one arena interval (group padding inside it belongs to no tile's valid part and is skipped).
    const size_t last = static_cast<size_t>(last_tensor);
    Span s;
    s.s0 = h.tensor_seg[static_cast<size_t>(first_tensor)];
    s.s1 = h.tensor_seg[last] + (h.tensor_n[last] > 0 ? 1 : 0);
    if (s.s1 <= s.s0) return MGWFBP_OK;                           // only empty tensors
    const size_t end_layer = static_cast<size_t>(h.seg_layer[static_cast<size_t>(s.s1 - 1)]);
    s.clipped = true;
    s.lo = static_cast<int64_t>(h.seg_off[static_cast<size_t>(s.s0)]);
    s.hi = static_cast<int64_t>(h.seg_off[static_cast<size_t>(s.s1 - 1)] + h.tensor_n[end_layer]);
    s.t0 = static_cast<int32_t>(s.lo / TILE);
    s.t1 = static_cast<int32_t>((s.hi + TILE - 1) / TILE);
    return run<K_PACK>(c, 0, d_grad_ptrs, d_merge_bufs, nullptr, nullptr, nullptr, 0.f, 0.f, hip_stream, &s);
}

int mgwfbp_reduce(mgwfbp_ctx* c, int32_t group, const void* const* d_merge_bufs, float* d_reduced,
                  void* hip_stream) {
    return run<K_REDUCE>(c, group, nullptr, const_cast<void* const*>(d_merge_bufs), d_reduced, nullptr, nullptr,
                         0.f, 0.f, hip_stream);
}

int mgwfbp_unpack_update(mgwfbp_ctx* c, int32_t group, const float* d_reduced, float* const* d_w_ptrs,
                         float* const* d_v_ptrs, float lr, float momentum, void* hip_stream) {
    return run<K_UPDATE>(c, group, nullptr, nullptr, const_cast<float*>(d_reduced), d_w_ptrs, d_v_ptrs, lr,
                         momentum, hip_stream);
}

int mgwfbp_reduce_update(mgwfbp_ctx* c, int32_t group, const void* const* d_merge_bufs, float* const* d_w_ptrs,
                         float* const* d_v_ptrs, float lr, float momentum, void* hip_stream) {
    return run<K_REDUCE_UPDATE>(c, group, nullptr, const_cast<void* const*>(d_merge_bufs), nullptr, d_w_ptrs,
                                d_v_ptrs, lr, momentum, hip_stream);
}

int mgwfbp_group_pipeline(mgwfbp_ctx* c, int32_t group, const void* const* d_grad_ptrs, void* const* d_merge_bufs,
                          float* d_reduced, float* const* d_w_ptrs, float* const* d_v_ptrs, float lr,
                          float momentum, void* hip_stream) {
    return run<K_PIPELINE>(c, group, d_grad_ptrs, d_merge_bufs, d_reduced, d_w_ptrs, d_v_ptrs, lr, momentum,
                           hip_stream);
}

int mgwfbp_group_pipeline_span(mgwfbp_ctx* c, int32_t group_first, int32_t group_count,
                               const void* const* d_grad_ptrs, void* const* d_merge_bufs, float* d_reduced,
                               float* const* d_w_ptrs, float* const* d_v_ptrs, float lr, float momentum,
                               void* hip_stream) {
    if (c == nullptr || !c->on_device) return MGWFBP_EINVAL;
    if (group_first < 0 || group_count < 0 || group_first > c->host.G - group_count) return MGWFBP_EINVAL;
    const Span s = span_of_groups(c->host, group_first, group_first + group_count);
    return run<K_PIPELINE>(c, 0, d_grad_ptrs, d_merge_bufs, d_reduced, d_w_ptrs, d_v_ptrs, lr, momentum,
                           hip_stream, &s);
}

int mgwfbp_group_pipeline_static(mgwfbp_ctx* c, int32_t group, const void* const* d_grad_ptrs,
                                 void* const* d_merge_bufs, float* d_reduced, float* const* d_w_ptrs,
                                 float* const* d_v_ptrs, float lr, float momentum, void* hip_stream) {
    if (c == nullptr) return MGWFBP_EINVAL;
    const HostTables& h = c->host;
    if (group < -1 || group >= h.G) return MGWFBP_EINVAL;
    auto round256 = [](size_t x) { return (x + 255) & ~static_cast<size_t>(255); };
    const size_t b_tiles = h.tiles.size() * sizeof(TileHdr);
    const size_t needed = round256(b_tiles) + round256(h.seg_n.size() * sizeof(uint32_t)) +    // the documented limit
                          round256(h.seg_layer.size() * sizeof(int32_t)) + round256(h.seg_off.size() * sizeof(uint64_t));
    if (needed > MGWFBP_STATIC_TABLE_MAX_BYTES) return MGWFBP_ECAPACITY;
    if (h.tiles.empty()) return MGWFBP_OK;

    int dev = -1;
    int rc = note(hipGetDevice(&dev));
    if (rc != MGWFBP_OK) return rc;
    if (dev < 0 || dev >= MAX_STATIC_DEVICES) return MGWFBP_EINVAL;
    std::lock_guard<std::mutex> lock(g_static_mutex);
    StaticSlot& slot = g_static[dev];
    if (slot.ptr == nullptr) {                    // first call on this device: where does its copy live?
        void* p = nullptr;
        rc = note(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (rc != MGWFBP_OK) return rc;
        if (p == nullptr) return MGWFBP_EHIP;
        slot.ptr = static_cast<unsigned char*>(p);
    }
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    if (!(slot.loaded && slot.serial == c->serial && slot.stream == stream)) {
        // The array still holds the previous call's tables: overwrite them, in stream order, with this model's.
        slot.loaded = false;
        rc = note(hipMemcpyAsync(slot.ptr, h.seg_block.data(), h.seg_block.size(), hipMemcpyHostToDevice, stream));
        if (rc != MGWFBP_OK) return rc;
        rc = note(hipMemcpyAsync(slot.ptr + h.seg_block.size(), h.tiles.data(), b_tiles, hipMemcpyHostToDevice, stream));
        if (rc != MGWFBP_OK) return rc;
        slot.loaded = true;
        slot.serial = c->serial;
        slot.stream = stream;
    }
    return run<K_PIPELINE>(c, group, d_grad_ptrs, d_merge_bufs, d_reduced, d_w_ptrs, d_v_ptrs, lr, momentum,
                           hip_stream, nullptr, reinterpret_cast<const TileHdr*>(slot.ptr + h.seg_block.size()));
}

int mgwfbp_handler_replay(mgwfbp_ctx* c, const double* group_ready_s, double time_scale,
                          int32_t max_groups_per_launch, void* const* streams, int32_t n_streams, const void* const* d_grad_ptrs, void* const* d_merge_bufs,
                          float* d_reduced, float* const* d_w_ptrs, float* const* d_v_ptrs, float lr, float momentum,
                          double* stats_out) {
    if (c == nullptr || !c->on_device || streams == nullptr || n_streams < 1 || n_streams > 16) return MGWFBP_EINVAL;
    if (!std::isfinite(time_scale) || time_scale < 0.0 || max_groups_per_launch < 0) return MGWFBP_EINVAL;
    const int32_t G = c->host.G;
    if (G > 0 && group_ready_s == nullptr) return MGWFBP_EINVAL;
    for (int32_t k = 0; k < G; ++k) {
        if (!std::isfinite(group_ready_s[k]) || group_ready_s[k] < 0.0) return MGWFBP_EINVAL;
        if (k > 0 && group_ready_s[k] < group_ready_s[k - 1]) return MGWFBP_EINVAL;
    }
    // Back-pressure for the batching forms: at most two launches queued per stream.  While a stream's earlier
    // launches are still running the GPU has work anyway, so the handler keeps collecting groups instead of
    // queueing ever more small launches behind them.  (One event per queue slot; created and destroyed here.)
    constexpr int DEPTH = 2;
    const bool throttle = max_groups_per_launch != 1;
    hipEvent_t slot_done[16 * DEPTH] = {};
    int rc = MGWFBP_OK;
    if (throttle) {
        for (int32_t j = 0; j < n_streams * DEPTH && rc == MGWFBP_OK; ++j)
            rc = note(hipEventCreateWithFlags(&slot_done[j], hipEventDisableTiming));
    }
    typedef std::chrono::steady_clock Clock;
    const Clock::time_point t0 = Clock::now();
    auto since_t0 = [&]() { return std::chrono::duration<double>(Clock::now() - t0).count(); };
    int32_t next = 0, launches = 0;
    while (next < G && rc == MGWFBP_OK) {
        const double due = time_scale * group_ready_s[next];
        double now = since_t0();
        while (now < due) now = since_t0();       // the backward pass has not produced this group yet
        const int32_t j = launches % n_streams;
        const int32_t slot = j * DEPTH + (launches / n_streams) % DEPTH;
        if (throttle && launches >= n_streams * DEPTH) {
            hipError_t q;
            while ((q = hipEventQuery(slot_done[slot])) == hipErrorNotReady) {
            }
            if (q != hipSuccess) {
                rc = note(q);
                break;
            }
            now = since_t0();
        }
        int32_t upto = next + 1;                  // everything that filled meanwhile goes into the same launch
        while (upto < G && time_scale * group_ready_s[upto] <= now &&
               (max_groups_per_launch == 0 || upto - next < max_groups_per_launch)) ++upto;
        const Span s = span_of_groups(c->host, next, upto);
        rc = run<K_PIPELINE>(c, 0, d_grad_ptrs, d_merge_bufs, d_reduced, d_w_ptrs, d_v_ptrs, lr, momentum,
                             streams[j], &s);
        if (rc == MGWFBP_OK && throttle) rc = note(hipEventRecord(slot_done[slot], static_cast<hipStream_t>(streams[j])));
        ++launches;
        next = upto;
    }
    // Drain every stream, also after a failed launch.  The handler thread has nothing else to do, so it polls
    // (a blocking wait sleeps, and waking up costs tens of microseconds per stream) and then confirms.
    for (int32_t j = 0; j < n_streams; ++j) {
        hipStream_t sj = static_cast<hipStream_t>(streams[j]);
        while (hipStreamQuery(sj) == hipErrorNotReady) {
        }
        const int rj = note(hipStreamSynchronize(sj));
        if (rc == MGWFBP_OK) rc = rj;
    }
    const double done = since_t0();
    for (hipEvent_t e : slot_done)
        if (e != nullptr) (void)hipEventDestroy(e);
    if (stats_out != nullptr) {
        const double last = G > 0 ? time_scale * group_ready_s[G - 1] : 0.0;
        stats_out[0] = static_cast<double>(launches);
        stats_out[1] = last;
        stats_out[2] = done;
        stats_out[3] = done - last;
    }
    return rc;
}

int mgwfbp_direct_update(mgwfbp_ctx* c, int32_t group, const void* const* d_grad_ptrs, float* d_reduced,
                         float* const* d_w_ptrs, float* const* d_v_ptrs, float lr, float momentum,
                         void* hip_stream) {
    return run<K_DIRECT>(c, group, d_grad_ptrs, nullptr, d_reduced, d_w_ptrs, d_v_ptrs, lr, momentum, hip_stream);
}

int mgwfbp_last_hip_error(void) { return g_last_hip_error; }

const char* mgwfbp_version(void) { return "mgwfbp-gfx950 0.1"; }

}  // extern "C"
