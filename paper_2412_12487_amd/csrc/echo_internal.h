// echo_internal.h -- device data layout and kernel launchers of libecho.so.
//
// The loader first cuts every (rank, stream) into segments: runs of compute and
// memcpy ops in which each op's only predecessor is the one before it and nothing
// else waits for an op inside the run.  A segment starts when its first op may and
// then runs for the sum of its ops' durations, so the composer's sweep walks
// segments instead of ops; the ops' own times are prefix sums from the segment's
// start, written by a parallel kernel after the last sweep.
//
// The sweep follows one "walk list" per walker: a walker is a group of consecutive
// ranks (one rank unless the graph has more ranks than the device holds co-resident
// wavefronts), and its list holds their segments and comm ops ordered by (key, rank,
// program order) where key is the first op's topological level in the merged graph (a
// collective merged into one barrier node) -- for a comm op, the level at which it can
// launch.  A wavefront walks one walker for 64 scenarios (one lane each); predecessors
// that are the latest op of a register slot stay in registers, the rest are read back
// from the finish array.  Collective barriers are met through per-(collective,
// scenario) arrival maxima and per-(collective, scenario tile) arrival counts, through
// member slots, or in LDS when every member sits in one workgroup.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "echo.h"

namespace echo {

constexpr int kStreams = 8;
constexpr int kClasses = 8;
constexpr int kTypes = 4;
constexpr int kLanes = 64;                       // scenarios per wavefront
constexpr int64_t kTimeLimit = int64_t(1) << 62;

// Device status bits (per graph).
constexpr unsigned kStatusRange = 1u;            // scenario knob out of range
constexpr unsigned kStatusOverflow = 2u;         // a time reached 2^62
constexpr unsigned kStatusTimeout = 4u;          // a barrier wait exceeded the spin limit
constexpr unsigned kStatusAbort = 8u;            // stop all waits (set with timeout)

// Ops of a segment, at most.  Longer runs are cut into consecutive segments: 32 keeps
// the parallel kernels' units even (two segments fill a 64-record chunk) while the sweep
// already skips nearly every op of the GPT graphs' runs of 8 to 30 ops.
constexpr int kSegOps = 32;

// One op of a segment (16 bytes); the records of a segment are contiguous, in order.
struct SegRec {
    int32_t op;
    uint32_t meta;      // class | kRecCompute | kRecFirst | kRecLast | kRecCand
    int64_t dur;        // base duration
};
static_assert(sizeof(SegRec) == 16, "segment record must stay 16 bytes");
constexpr uint32_t kRecCompute = 8u;     // a compute op (else memcpy: never inflated)
constexpr uint32_t kRecFirst = 16u;      // first op of its segment
constexpr uint32_t kRecLast = 32u;       // last op of its segment
constexpr uint32_t kRecCand = 64u;       // on a first op: overlap detection looks at the segment

// One entry of a walk list (32 bytes, read wave-uniformly): a segment or a comm op.
// The (rank, stream) pairs of a walker are mapped to eight register "slots": slot 0
// is its busiest compute/memcpy stream, so most items only touch slot 0.  Pairs
// left without a slot (a walker of several ranks) keep nothing in registers:
// their ops carry kNoReg and their successors read them back from memory.
// A comm op's launch item publishes its arrival; a resolve item placed right
// before its first successor waits for the barrier and writes its finish (to its
// slot, or only to memory without one).
struct WalkItem {
    int32_t op;         // op id: row of the [op][scenario] outputs (a segment: its first op)
    uint32_t meta;      // kind | slot << 2 | regmask << 8 | has far << 16 | noreg << 17
                        // | linked << 18 | need finish << 19 | fold << 20 | launch << 21
                        // | empty << 31
    int32_t far_off;    // predecessors read back from memory: far[far_off .. +nfar)
    int32_t coll;       // segment: its last op.  Comm op: its collective; of a collective met
                        // by counting arrivals in device memory (neither in LDS nor through
                        // member slots), its index among those collectives
    int64_t dur;        // sum of a segment's base durations; resolve item: cost class
    int32_t nfar;
    int32_t aux;        // segment: number of ops
};
static_assert(sizeof(WalkItem) == 32, "walk item must stay 32 bytes");

// The item has predecessors to read back from memory.
constexpr uint32_t kHasFar = 1u << 16;
// The op's (rank, stream) pair has no register slot.
constexpr uint32_t kNoReg = 1u << 17;
// Comm op linked to the comm op before it on its stream: the launch item publishes a launch
// time that leaves that op's finish out (and stores it in the start row), the resolve item
// takes the finish from the stream's slot (without one, from the row of op nfar) and
// applies it.
constexpr uint32_t kLinked = 1u << 18;
// The op's finish is read as a far predecessor: stored also by a pass that stores nothing
// else (the last one, when neither timelines nor digests are asked for).
constexpr uint32_t kNeedF = 1u << 19;
// Resolve item: after writing the comm op's finish, raise slot 0 to it.  Among the items
// folded before one segment, slot 0's own comm ops come first (they set slot 0).
constexpr uint32_t kFold = 1u << 20;
// Resolve item of a collective met in LDS that also is the comm op's launch, at slot 0's
// value: the launch item right before it, waiting for nothing but the latest op of slot 0,
// left out (a blocking all-reduce after a segment).
constexpr uint32_t kLaunch = 1u << 21;
// Padding at the end of a round.
constexpr uint32_t kEmpty = 1u << 31;
// Item kind (besides compute/comm/memcpy) that finishes a comm op:
// wait for its barrier, then write its finish.
constexpr int kResolve = 3;

// Workgroups walk kBlockWalkers consecutive walkers (one wavefront each) for
// one scenario tile.  A collective whose members all sit in one block is met in
// LDS: each communicator of the block owns a channel with two alternating
// slots (max of launch times per lane, arrival count).  Collective costs are
// looked up per cost class -- the (type, S, N, M, K) tuple that fixes T(c, s)
// for a scenario -- and a block stages its most used classes in LDS.
constexpr int kBlockWalkers = 8;
constexpr int kFlagRowTiles = 2;    // a final mask pass of this many tiles per launch is labelled kInMaskFlags
constexpr int kWalkersPerCu = 16;   // wavefronts of a walk launch per compute unit, at most
// A walk list is cut into rounds of kBlock items (padded with empty ones) of which at most
// kDurs are segments: a round's items and its segments' durations are fetched a round ahead,
// into registers that the loop over the round's items only reads.  (A register written
// inside that loop while its load is in flight is copied at every join of the loop's
// branches, and each copy waits for the load: with the durations refilled inside the loop,
// eight at a time, the refined pass of a 96-rank job took 7.4 instead of 4.7 ms.)
constexpr int kBlock = 32;
constexpr int kDurs = 8;
constexpr int kChannels = 8;          // LDS barrier channels per block
constexpr int kClassSlots = 8;        // LDS cost classes per block
constexpr uint32_t kNoSlot = 15;
// Comm item aux word: bit 0 local barrier | slot parity << 1 | channel << 2 |
// class slot << 5 (kNoSlot: read the class's cost from global memory) | expected count << 9.
constexpr uint32_t kAuxLocal = 1u;
constexpr int kExpectedBits = 23;
// A collective met in device memory whose members are few (at most kSlotMembers)
// meets through per-member slots: each member's launch item stores its launch time
// into its own slot (cleared to -1 before every pass), and a resolve item reads all
// its collective's slots -- a value of -1 means "not yet launched".  The launch item
// carries its slot in `dur`, the resolve item the collective's first slot in
// `far_off`; aux bit 1 (without bit 0) marks the mode and the expected-count field holds the member
// count.  Larger collectives count their arrivals and keep a per-scenario maximum.
constexpr uint32_t kAuxSlots = 2u;
constexpr int kSlotMembers = 8;
__host__ __device__ inline uint32_t aux_local(int channel, int parity) {
    return kAuxLocal | ((uint32_t)parity << 1) | ((uint32_t)channel << 2);
}
__host__ __device__ inline int aux_barrier(uint32_t x) { return int((x >> 1) & 15u); }   // channel * 2 + parity
__host__ __device__ inline int aux_slot(uint32_t x) { return int((x >> 5) & 15u); }
__host__ __device__ inline unsigned aux_expected(uint32_t x) { return x >> 9; }

__host__ __device__ inline int item_kind(uint32_t m) { return int(m & 3u); }
__host__ __device__ inline int item_stream(uint32_t m) { return int((m >> 2) & 7u); }
__host__ __device__ inline unsigned item_regmask(uint32_t m) { return (m >> 8) & 0xffu; }

// Overlap detection records, per compute op and scenario, which collective
// types overlap it as a 4-bit mask (bit t: some comm op of type t on the same
// rank overlaps).  The slowdown factor is the largest table entry
// slowdown_q16[class][t] over the set bits, 65536 for an empty mask.
//
// A segment it looks at (32 bytes), and per comm stream of the rank the comm ops that
// may overlap it: positions [lo, hi) of the stream's list.  Those before lo finish before
// the segment can start (one of them is a predecessor of an op of its stream up to its
// first), those from hi on launch after its last op (some op from it on in its stream is
// a predecessor).  Segments without any such comm op overlap nothing and have no entry.
struct OverlapSeg {
    int32_t rec0, n;        // its records
    int32_t first, last;    // its first and last op
    int32_t cand0, ncand;   // its ranges of comm ops
    int32_t pad[2];
};
static_assert(sizeof(OverlapSeg) == 32, "overlap segment must stay 32 bytes");
struct CommRange {
    int32_t lo, hi;         // positions in the comm lists
    int32_t last_op;        // the comm op at hi - 1
    int32_t seg;            // its overlap segment
};
static_assert(sizeof(CommRange) == 16, "comm range must stay 16 bytes");
// segments a wavefront of overlap detection takes at a time (their ranges, at most eight
// each, fit the lanes)
constexpr int kOverlapGroup = 8;

// First and last op of a segment: the rows its start and finish live in.
struct RowPair {
    int32_t first, last;
};

// Chunk of segment records, the unit of the kernels that sum durations and write
// timelines: whole segments, at most 64 records (one vector load).
struct RecChunk {
    int32_t rec0, cand0;    // first record; overlap segments before it
};

// Inputs of the CC model for a table of collectives (or of cost classes).
struct CollTable {
    int64_t n = 0;
    int64_t *bytes = nullptr;        // S
    int64_t *chunk = nullptr;        // chunk size (Table 6)
    int64_t *eta_ring = nullptr;     // ceil(S / (N * chunk))
    int64_t *eta_chunks = nullptr;   // ceil(S / chunk)
    int32_t *N = nullptr, *M = nullptr, *K = nullptr;
    uint8_t *type = nullptr;
    // cost classes only, to cost every collective through its class: class k's cost goes to
    // row row[k] (its first collective) of n_out rows, and from there to the row of every
    // other collective c of class class_of[c]
    int32_t *row = nullptr, *class_of = nullptr;
    int64_t n_out = 0;
};

// Device copy of a loaded graph (all pointers are device memory).
// Device form of a tree node, one 16-byte load: the two children of a split sit side
// by side, and the walk goes to left + (x >= threshold).  A leaf loops to itself
// (threshold INT64_MIN, left = its own index - 1), so every tree is walked exactly
// ECHO_TREE_DEPTH steps without a branch; leaf values live in a separate array.
struct DevTreeNode {
    int64_t threshold;
    int32_t feature;
    int32_t left;
};
static_assert(sizeof(DevTreeNode) == 16, "one 16-byte load per node");

// Compact form of the ensemble, held in LDS while overlap detection runs.  Features are
// compared by bin: for feature f the ensemble's split thresholds, sorted and without
// repeats, are T_f[0 .. K_f); the bin of a value x is the number of them <= x, so
// "x < T_f[r]" holds exactly when bin(x) <= r.  A node is one 32-bit word laid out like
// DevTreeNode (breadth first per tree, a split's children side by side): feature
// (bits 0-3), the rank r of its threshold in T_f (bits 4-17), left child minus its own
// index (bits 18-31; right = left + 1).  A leaf has feature kFxLeaf and its value in
// bits 4-31 (signed); its feature's bin is always 0, so it loops to itself.
constexpr int kFxFeatures = 12;
constexpr uint32_t kFxLeaf = 15;
constexpr int kFxRows = 16;                  // bin rows per lane; rows 12..15 stay 0
constexpr int kFxMaxWords = 12 * 1024;       // LDS budget of the nodes (48 KB of a 64 KB workgroup, roots aside)
constexpr int kFxRankBits = 14;
struct CompactForest {
    uint32_t *words = nullptr;               // [n_words]
    int32_t n_words = 0;                     // 0: no compact form (the ensemble does not fit)
    int64_t *thr = nullptr;                  // every feature's thresholds, concatenated
    int32_t thr_off[kFxFeatures + 1] = {};   // feature f: thr[thr_off[f] .. thr_off[f + 1])
    int32_t *cbin = nullptr;                 // [class][kFxFeatures]: bins of the class's own features
    int32_t tbin[4] = {};                    // bin of each collective type
    int32_t *coll_bin = nullptr;             // [coll][2]: bins of S and of the N its cost uses
    int32_t *cp_bin = nullptr;               // [segment record]: bin of the base duration
};

struct DeviceGraph {
    int64_t n_ops = 0, n_colls = 0;
    int32_t n_ranks = 0, n_walkers = 0, n_blocks = 0;
    WalkItem *items = nullptr;       // walk lists, walker-major
    int64_t *round_off = nullptr;    // [n_walkers + 1] rounds of each walker: kBlock items, kDurs rows each
    int32_t *walk_rows = nullptr;    // last op of the rounds' segments
    int32_t *walk_recs = nullptr;    // their first records
    RowPair *far = nullptr;          // far predecessors: a segment's first and last op, or a comm op (first -1)
    CollTable colls;                 // every collective
    int32_t *members = nullptr;      // [n_colls] member ops present: arrivals that complete a barrier
    CollTable classes;               // every cost class
    int32_t *block_class = nullptr;  // [n_blocks][kClassSlots] class staged in each LDS slot, -1 = none
    // segments: their ops, and the chunks of records
    SegRec *recs = nullptr;
    RecChunk *chunks = nullptr;      // [n_chunks + 1]
    int64_t n_recs = 0, n_chunks = 0;
    // overlap detection: the segments it looks at, and the comm ops of each (rank, stream)
    // in program order
    OverlapSeg *osegs = nullptr;
    CommRange *ranges = nullptr;
    int64_t n_osegs = 0;
    int32_t *cl = nullptr;
    uint8_t *cl_type = nullptr;      // collective type of each listed comm op
    unsigned *status = nullptr;      // device status word
    echo_cc_table *cc_tables = nullptr;   // CC parameter tables (echo_set_cc_tables)
    int32_t n_cc_tables = 0;
    int32_t *cl_coll = nullptr;      // collective of each listed comm op (parallel to cl)
    // slowdown ensemble (echo_set_forest)
    DevTreeNode *forest_nodes = nullptr;
    int32_t *forest_leaf = nullptr;  // [node] value of a leaf (0 for a split)
    int32_t *forest_roots = nullptr;
    int64_t *class_metrics = nullptr;  // [8][4]
    int32_t n_trees = 0, forest_base = 65536;
    CompactForest fx;                  // the ensemble in LDS form, when it fits
    int32_t max_ranges = 0;          // the most comm ranges of one overlap segment
    int64_t n_slots = 0;             // member slots of the collectives met through slots
    int64_t n_counted = 0;           // collectives met by counting arrivals in device memory
    int32_t *counted_members = nullptr;   // [n_counted] their member ops present
};

constexpr int kClassMetrics = 4;

// One pass over a range of scenario tiles: in the first pass the segments' jittered
// durations are summed, then the sweep, and after the last one the ops' times.
//
// Between the passes the finish row of a segment's last op holds the segment's duration:
// k_sum puts it there (the first pass of a tile with jitter) or the first sweep (a tile
// without, whose durations are the items'), and overlap detection changes it; the last
// sweep replaces it by the finish.
struct WalkArgs {
    const WalkItem *items;
    const int64_t *round_off;        // [walker + 1]
    const int32_t *rows;             // [round][kDurs] last op of its segments
    const RowPair *far;
    const int32_t *c_N;              // [counted coll] member ops present (arrivals that complete the barrier)
    const int32_t *block_class;
    const echo_scenario *scen;
    const int64_t *class_cost;       // [class][scen]
    const SegRec *recs;
    const RecChunk *chunks;
    int64_t n_chunks;
    // Per-op outputs of overlap detection, one row per segment record of a flagged segment,
    // mstride columns (the tiles' scenarios, padded to whole tiles):
    const uint8_t *tmask;            // overlap type masks, or null
    const uint32_t *ext;             // extra times (prorating, ensemble factors), or null
    const uint8_t *xflag;            // [overlap segment][tile]: nonzero when some mask (extra time) of it is
    int64_t mstride;
    const unsigned *stable;          // non-null: skip the pass when *stable (every scenario at its fixed point)
    int64_t *start, *finish;         // [op][scen]
    unsigned long long *arrive;      // [counted coll][scen] latest member launch
    unsigned *count;                 // [counted coll][tile] members arrived
    int64_t *slots;                  // [slot][scen] launch time of a slot collective's member, -1 before it
    int64_t *step;                   // [scen]
    uint64_t *digest;                // [scen] or null
    unsigned *status;
    int64_t spin_limit;              // wall-clock ticks (100 MHz) before a wait gives up
    int32_t n_scen, n_tiles;
    int32_t tile0, tiles;            // tiles handled by this launch
    int32_t n_walkers;
    int32_t in;                      // what the pass is refined by (kIn*)
    int32_t final_pass;              // accumulate step time (and digest)
    int32_t timelines;               // final pass: write every op's start and finish
    // kInOps only, and last: among the fields above they moved the argument loads of every
    // variant (a fixed point's sweeps took 2 % longer)
    const int32_t *rec_rows;         // [round][kDurs] first records of the round's segments
    int64_t n_recs;
};


struct OverlapArgs {
    const OverlapSeg *osegs;
    const CommRange *ranges;
    int64_t n_osegs;
    const SegRec *recs;
    const int32_t *cl;
    const uint8_t *cl_type;
    const echo_scenario *scen;
    const int64_t *start;            // the previous pass's times
    int64_t *finish;                 // of comm ops: their finishes; of segments (last op): in/out their durations
    // rows of the segment records, mstride columns
    uint8_t *tmask;                  // in: masks of the previous pass (if it was refined), out: new ones
    uint32_t *ext;                   // prorating: in/out like tmask, the extra time q16(o, F) - o
    uint8_t *xflag;                  // in/out, [overlap segment][tile]: nonzero when some mask (extra time) of it is
    int64_t mstride;
    unsigned *chg;                   // non-null: [scen] set when some duration changes
    const unsigned *stable;          // non-null: skip when *stable
    // ensemble factors (forest_nodes non-null): features of the overlapping comm ops
    const int32_t *cl_coll;
    const int64_t *coll_bytes;       // S of each collective
    const int32_t *coll_N;           // N its cost uses
    const DevTreeNode *forest_nodes;
    const int32_t *forest_leaf;
    const int32_t *forest_roots;
    const int64_t *class_metrics;
    int32_t n_trees, forest_base;
    CompactForest fx;                // n_words > 0: the compact ensemble (LDS variant)
    int32_t prorate;                 // inflate only the overlapped part (extra times in ext)
    int32_t n_scen, n_tiles;
    int32_t prev_refined;            // the previous pass inflated its compute ops
    unsigned *status;
};

// Kernel launchers (echo_kernels.hip).  All enqueue on `stream`.
hipError_t launch_init(const DeviceGraph &g, const echo_scenario *scen, int32_t n_scen,
                       unsigned long long *arrive, int64_t n_arrive, unsigned *count,
                       int64_t n_count, int64_t *slots, int64_t n_slot_values, int64_t *step,
                       uint64_t *digest, hipStream_t stream);
hipError_t launch_clear(unsigned long long *arrive, int64_t n_arrive, unsigned *count,
                        int64_t n_count, int64_t *slots, int64_t n_slot_values, hipStream_t stream);
hipError_t launch_cc_cost(const CollTable &t, const echo_cc_table *tables, const echo_scenario *scen,
                          int32_t n_scen, int64_t *cost, unsigned *status, hipStream_t stream);
hipError_t launch_walk(const WalkArgs &a, int32_t n_blocks, hipStream_t stream);
// max_ranges: the most comm ranges of one segment (selects the kernel variant)
hipError_t launch_overlap(const OverlapArgs &a, int32_t max_ranges, hipStream_t stream);
// Bins of the compact ensemble's per-collective (S, N) and per-record (base duration)
// features.
hipError_t launch_forest_bins(const DeviceGraph &g, int64_t n_compute, const CompactForest &fx,
                              hipStream_t stream);
// After an overlap pass: count the refinement of every scenario whose durations changed,
// clear the change flags, and set *stable when none changed.
hipError_t launch_settle(unsigned *chg, int32_t n_scen, int32_t *refinements, unsigned *stable,
                         hipStream_t stream);
// Fill n int32 with v (a kernel, so the sequence stays capturable).
hipError_t launch_fill_i32(int32_t *p, int64_t n, int32_t v, hipStream_t stream);
// What a pass is refined by, the walk kernel's first template argument.  The sweep itself
// only tells the first pass from the others; the rest is a label that keeps the passes
// apart in kernel traces: refined by masks (a final pass over many tiles, whose timelines
// fill the memory system, under a name of its own) or by extra times.  With kInOps the
// sweep draws every op and writes its times itself, without k_sum and k_expand.
constexpr int kInNone = 0;        // first pass: base durations
constexpr int kInMasks = 1;       // overlap masks
constexpr int kInMaskFlags = 2;   // overlap masks, final pass of kFlagRowTiles tiles per launch or more
constexpr int kInExtFlags = 3;    // prorated or ensemble extra times
constexpr int kInOps = 4;         // only pass (no refinement, no digest): the sweep walks the segments' ops
inline int walk_input(bool refined, bool ext, bool many_tiles) {
    return !refined ? kInNone : ext ? kInExtFlags : many_tiles ? kInMaskFlags : kInMasks;
}
// Co-resident walk workgroups (kBlockWalkers wavefronts each) the device can hold,
// for each kernel variant (bits 0-2 input, bit 3 final, bit 4 digest); at most
// kWalkersPerCu / kBlockWalkers per compute unit.
constexpr int kWalkVariants = 32;
hipError_t walk_capacity(int device, int64_t workgroups[kWalkVariants]);
inline int walk_variant(int in, bool final_pass, bool digest) {
    return in | (final_pass ? 8 : 0) | (digest ? 16 : 0);
}
// Device address of this GPU's fixed workspace array (ECHO_SCRATCH_BYTES) for
// echo_compose_batch_static; `device` must be current.  Looked up once per device.
hipError_t scratch_buffer(int device, void **ptr);
// Largest prorated extra time an op may carry (its staging slot is 32 bits).
constexpr uint32_t kExtLimit = 0xFFFFFFFFu;

}  // namespace echo
