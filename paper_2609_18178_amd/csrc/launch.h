// launch.h -- internal interface between the host validation layer
// (pactshard.hip) and the gfx950 kernels (kernels.hip).  Not installed.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace pact {

// Segments handled by one kernel launch; longer tables take several launches.
// The batch travels in the kernel-argument segment (about 2 KB), so no device
// table has to be allocated or copied.
constexpr int kSegsPerLaunch = 32;

// Threads per workgroup (4 waves of 64).
constexpr int kBlock = 256;

// The stream probe's tile: four 16-byte vectors of fp32 elements per thread and
// array, 4096 elements.  Also the tile that the limit on a shard's size is stated in.
constexpr int kVec = 4;
constexpr int kUnroll = 4;
constexpr int kTile = kBlock * kVec * kUnroll;

// A dispatch counts its work-items in 32 bits, so one launch holds at most
// this many tiles.
constexpr uint64_t kMaxTiles = UINT32_MAX / kBlock;

// Digest partial sums: each result slot owns kLanes workspace lines of
// kLaneStride words (256 bytes); a line begins with kNodesPerLane nodes of two
// words: two sets each of a lane's node, of a slot's own (in lane 0's line; the
// total's in lane 1's of slot 0) and of the total's lanes (of slot 0).
constexpr int kLanes = 16;
constexpr int kLaneStride = 32;
constexpr int kNodesPerLane = 6;

// Tiles whose arrivals the nodes of one result can count: 2^20 per lane.
constexpr uint64_t kGatherTiles = (uint64_t)kLanes << 20;

// Where the tiles' shares go.
struct Results {
    uint64_t* digest;      // result slots
    uint64_t* words;       // the workspace, or null: shares are added to the result slots
    uint32_t set;          // which set of nodes the call uses (0 or 1)
    uint32_t total_slot;   // the slot of the per-segment results' sum
    uint32_t total_tiles;  // the call's tiles, which also gather into total_slot; 0: they do not
};

// Per-segment binary32 scalars of one step.
struct StepScalars {
    float beta1, beta2, eps, decay, omb1, omb2, step_size, rs_bc2;
};

// A segment whose arrays are nowhere 16-byte (fp32 and BF16 state) and 8-byte
// (bf16 copy) aligned at the same element.
constexpr uint32_t kNeverAligned = ~0u;

// One segment of a launch: a line of 64 bytes, so that a tile's workgroup waits
// for one.  It owns the tiles [tile_begin, tile_end), at least one (an empty
// segment's tile hands in a share of zero): they cover its elements from the first
// aligned one on, and the first tile those before it.
struct alignas(64) Segment {
    uint64_t elem_begin;  // shard-relative first element
    uint64_t elem_count;
    uint32_t tile_begin, tile_end;
    uint32_t align;  // elements before the first aligned one, or kNeverAligned
    StepScalars sc;
};
static_assert(sizeof(Segment) == 64, "one line");

// One launch's slice of the segment table.  Tiles never straddle segments.
struct Batch {
    uint32_t nseg;
    uint32_t slot0;        // result slot of this batch's first segment
    uint32_t tile0;        // tiles of the call's earlier batches
    uint32_t tiles;        // of this batch
    uint32_t passes;       // passes of a tile
    uint32_t per_segment;  // nonzero: one result slot per segment, else one in all
    alignas(64) uint32_t tile_begin[kSegsPerLaunch];  // the segments', ~0 behind the last
    Segment seg[kSegsPerLaunch];
};

struct Arrays {
    float* p;
    const float* g;
    float* g_zero;      // the grad array, written only by Mode::CommitZeroGrad
    float* m;
    float* v;
    uint16_t* b;
    uint64_t goff;      // global flat index of shard element 0
    Results res;
};

// The same arrays for a shard held in BF16 (no separate working copy).
struct ArraysBf16 {
    uint16_t* p;
    const uint16_t* g;
    uint16_t* m;
    uint16_t* v;
    uint64_t goff;
    Results res;
};

enum class Mode : int {
    Commit = 0,
    StateDigest = 1,
    Bf16Digest = 2,
    CommitZeroGrad = 3,
    GradGuard = 4,
    CommitBf16State = 5,
    DigestBf16State = 6,
};

// A pass of a mode's tile kernel: `rows` rows of kBlock vectors of `vec`
// elements.  A tile is Batch::passes of them, one after the other.
struct Shape {
    int vec, rows;
    constexpr uint32_t elems() const { return (uint32_t)(kBlock * vec * rows); }
};

// The instantiations of a mode's tile kernel: the usual one, one for shards that
// would leave most of the GPU idle, and one with longer tiles.
enum class Form : int { Usual, Small, Long };

// The commits of binary32 state move one row of 4 KB per array (the comment at
// kReserveLds in kernels.hip says why), or four (Long; the state digest's Long tiles have
// several passes); the others' kernels, bound by
// reading or by VALU issue, have more loads in flight per thread, and a second shape of
// one short row for shards that would leave most of the GPU idle (Small).
constexpr Shape shape_of(Mode m, Form f) {
    const bool small = f == Form::Small;
    switch (m) {
        case Mode::Commit:
        case Mode::CommitZeroGrad:
            return f == Form::Long ? Shape{4, 4} : Shape{4, 1};
        case Mode::GradGuard:
            return {4, 4};
        case Mode::StateDigest:
            return small ? Shape{4, 1} : Shape{4, 4};
        case Mode::Bf16Digest:
        case Mode::CommitBf16State:
        case Mode::DigestBf16State:
            return small ? Shape{4, 1} : Shape{8, 2};
    }
    return {4, 1};
}

constexpr bool binary32_commit(Mode m) { return m == Mode::Commit || m == Mode::CommitZeroGrad; }
constexpr bool has_long(Mode m) { return binary32_commit(m) || m == Mode::StateDigest; }

// Elements up to which the small shape is the faster one (0: there is none).
// us per call, small / large shape, at 0.1M, 1M, 4M and 16M elements:
//   state digest  4.1 / 5.3   6.0 / 6.4  12.8 / 12.8  42.4 / 38.9
//   bf16 digest   3.6 / 3.6   4.9 / 4.5   8.6 / 6.0   22.0 / 13.5 (of 0.3M in 138 segments
//                 21.9 / 24.0)
//   BF16 digest   4.0 / 5.0   5.7 / 6.0  12.0 / 11.4  37.8 / 32.0
// and of the BF16 commit at 2M, 4M, 8M and 16M:
//                 9.3 / 10.2 14.4 / 16.0 23.6 / 24.9  43.7 / 44.9
constexpr uint64_t small_up_to(Mode m) {
    switch (m) {
        case Mode::StateDigest: return 3u << 20;
        case Mode::Bf16Digest: return 1u << 19;
        case Mode::CommitBf16State: return 16u << 20;
        case Mode::DigestBf16State: return 3u << 19;
        default: return 0;
    }
}

// State digests of this many elements and more hand in once for four passes.  Each
// hand-in holds a wave slot for the answer of an atomic, but long tiles leave the GPU
// emptier at the end.  us in tiles of one / four passes: 220M elements 438.4 / 442.0, 300M
// 597.9 / 599.2, 400M 797.1 / 797.4, 453M 905.4 / 901.4, 1800M 3612 / 3587.
constexpr uint64_t kLongDigestFrom = 3u << 27;
constexpr uint32_t kLongDigestPasses = 4;

// The form of a call over `elems` elements, `longest` of them in its longest segment.
// A segment's tiles have to fit one launch: where those of a binary32 commit do not (17e9
// elements), they are the longer ones, which the host's limit is stated in.  And without
// a workspace each tile adds its share to the one result word, 12 ns per tile whatever
// else the call does, so its tiles are the longest there are.  us per call of 1M and 453M
// elements without a workspace, in tiles of 1024 and of 4096 elements: commit 17.1 / 11.2
// and 5504 / 2420; of 1M and 3M, state digest 16.1 / 9.2 and 40.0 / 15.0; BF16 commit of
// 16M 196 / 64.
constexpr Form form_of(Mode m, uint64_t elems, uint64_t longest, bool workspace) {
    const bool longer = !workspace || longest / shape_of(m, Form::Usual).elems() >= kMaxTiles;
    if (longer) return binary32_commit(m) ? Form::Long : Form::Usual;
    if (m == Mode::StateDigest && elems >= kLongDigestFrom) return Form::Long;
    return elems <= small_up_to(m) ? Form::Small : Form::Usual;
}

// Consecutive tiles per XCD: a workgroup's XCD is its number modulo 8, so tiles
// are dealt in groups of 8 * run, of which each XCD takes `run` neighbours.
// Grids below `from` tiles keep their order.
struct Runs {
    uint32_t run, from;
    uint32_t long_run, long_from;
};
constexpr uint32_t kXcds = 8;
constexpr Runs runs_of(Mode m, Form f) {
    constexpr uint32_t kNever = ~0u;
    if (f != Form::Usual) return {1, kNever, 1, kNever};
    switch (m) {
        case Mode::Commit:
        case Mode::CommitZeroGrad:
            // Of 128 KB per array, and 512 KB where that leaves 32 groups: us per
            // commit in runs of 1 / 32 / 128 tiles: 83.7 / 79.8 / 83.2 at 16M
            // elements, 163 / 154 / 152 at 32M, 395 / 368 / 361 at 76M.
            return {32, 0, 128, 32768};
        case Mode::StateDigest:
            return {1, kNever, 1, kNever};  // bound by VALU issue: no difference
        default:
            // 16 tiles against 1: guard of 453M elements 288 -> 266 us, BF16
            // digest 728 -> 720, BF16 commit 1237 -> 1225; below 8M elements
            // up to 7% slower.
            return {16, 2048, 16, kNever};
    }
}

// The tile of a block, with runs of `run` tiles per XCD; the blocks behind the last
// whole group keep their order.
constexpr uint32_t dealt_tile(uint32_t block, uint32_t tiles, uint32_t run) {
    const uint32_t group = kXcds * run;
    const uint32_t r = block % group, first = block - r;
    return tiles - first >= group ? first + r % kXcds * run + r / kXcds : block;
}

// Enqueue the clearing of what the tile kernels hand their shares in to: the
// nodes of nres result slots when `words` is given, else the nslots digest slots.
hipError_t launch_clear(uint64_t* digest, uint64_t* words, uint32_t nres, uint32_t nslots, hipStream_t stream);

// Enqueue one batch in the given mode, in tiles of shape_of(mode, form): one
// workgroup per tile, so `grid` is the batch's tile count.
hipError_t launch_batch(Mode mode, Form form, const Arrays& a, const Batch& b, uint32_t grid, hipStream_t stream);

// Enqueue one batch of a BF16-state mode (CommitBf16State, DigestBf16State).
hipError_t launch_batch_bf16(Mode mode, Form form, const ArraysBf16& a, const Batch& b, uint32_t grid,
                             hipStream_t stream);

// Enqueue digest[nres] = sum of digest[0..nres).
hipError_t launch_total(uint64_t* digest, uint32_t nres, hipStream_t stream);

// Enqueue the 30-byte/element stream probe (n a multiple of kVec): one
// workgroup per tile when workgroups == 0, else a persistent grid of that
// many workgroups striding over the tiles.
hipError_t launch_probe(const float* i0, const float* i1, const float* i2, const float* i3,
                        float* o0, float* o2, float* o3, uint16_t* oh, uint64_t n, uint32_t workgroups,
                        hipStream_t stream);

}  // namespace pact
