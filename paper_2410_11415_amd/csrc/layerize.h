// Host-side layerization and tensorization of a circuit DAG (paper Section 3.1 Eq. 2,
// Section 3.2, Appendix C Alg. 2 and Alg. 3).  Pure C++, no device code: the result is a set
// of plain index arrays that the evaluator uploads once.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

namespace klay {

struct Options {
    bool no_reorder = false;
    int32_t heavy_fan = 48;     // rows with more sources than this are evaluated in split passes
    int32_t min_segment = 24;   // smallest segment of a split row, in edges
    bool no_tail = false;       // never use the persistent kernels for the narrow top layers
    bool alias_chains = false;  // no unary chain nodes below the narrow top of the circuit: edges index the rows of any lower layer
    bool no_merge = false;      // keep structurally identical gates apart
    int32_t tail_rows_cap = 0;  // > 0: layers with more nodes than this are no candidates for the persistent kernels
                                // (at most kTailRowsCap; for tests of the boundary between the two parts)
    bool small_batch_edges = false;   // evaluator option (not used by the layerizer): lanes = edges kernel for B <= 32
    bool no_fusion = false;     // build no fused plans (LayerPlan::fwd2): every forward sweep writes every AND node's value
};

// Layers at the top of the circuit with at most this many nodes are candidates for the persistent
// kernels, which keep two layers of one batch column in LDS (values forward, adjoints in the reverse sweep):
// 20000 rows is what two arrays in 160 KB hold.  The layers above alias_top have no row with more sources than kTailFanCap;
// the narrow layers of circuits with longer rows are a plan of their own (TopPlan), in which a layer has at most kTopEdges
// edges.
constexpr int64_t kTailRowsCap = 20000;
constexpr int64_t kTailFanCap = 64;
constexpr int64_t kTopEdges = 160000;
// With more stand-ins of leaves than this the first layer is left to the launches: from layer 1 on the kernels evaluate the leaves
// themselves and the reverse sweep has a row for every stand-in (8138 leaves, 23200 nodes in 30 layers, 120000 of these, us
// at B = 64: forward 100, training step 200; from layer 2 on 89 and 179; 1120 leaves and 22000 of these: 125 and 286 against
// 136 and 333).
constexpr int64_t kTopLeafStandIns = 100000;

// Waves of a workgroup of those kernels.
constexpr int kColWaves = 16;

// Index vectors of one layer in the form the persistent kernels walk: runs of consecutive rows of one kind, read in blocks of
// 64 lanes x 16 entries of 16 bits (32 bytes per lane in two lines of 1 KB).
//   Kinds 0, 1, 2: rows of at most 1, 2 or 4 entries, in chunks of 64 rows: a block holds 16, 8 or 4 chunks, row
// 64 i + lane of the run has the lane's entries from i << kind on.  Kinds 3, 4: units of 64 >> k rows, 2^k lanes
// per row (k chosen per run): lane j works for row j >> k and holds that row's entries (j mod 2^k) + i * 2^k, and the
// lanes of a row meet in a butterfly at the end.  A unit of kind 4 has at most 8 entries per lane (the first line of
// one block), one of kind 3 as many blocks as its run says.  A row of many entries
// therefore spreads over the wave instead of making 63 lanes wait for one; a row may have up to kColRowEntries entries.
//   An entry is an LDS slot (kColSlots + position of the source: the first slots of a value array hold the identities
// that padding names, kColPadAnd for AND layers and the reverse sweep, kColPadOr for OR layers).  Bit 15 is a flag of the
// reverse sweep: weighted edge, or (steps through an AND layer, on every entry of the row) the row's adjoint is
// stored in the one-gather form.  Slots stay below 2^15.
//   Descriptor of a run, 2 words: [0] LDS slot of its first row | blocks per unit << 15, [1] rows | k << 16 | kind << 20.
// The descriptors of a wave in a layer come in tables of 64: up to 63 runs and one of no rows (word 0 = 1: another
// table follows, 0: the end).  The rows of a layer are cut into chunks and units by a shortest-path search over their
// cost, and every wave gets a contiguous share of about the same cost, so that the waves reach the layer's barrier together.
//   The forward kernel has one wave less for this: its last wave moves the values to the column-major buffer.  So has
// the reverse kernel over a TopPlan: it moves the adjoints.
constexpr int kColSlots = 4, kColPadAnd = 0, kColPadOr = 1;
constexpr int kColFwdWaves = kColWaves - 1, kColBwdWaves = kColWaves, kTopBwdWaves = kColWaves - 1;
constexpr int kBlockWords = 512, kLineWords = 256, kDescWords = 2, kDescTable = 64;
constexpr int64_t kColBlocksMax = (1 << 17) - 1;             // blocks of a unit: what the descriptor holds
constexpr int64_t kColRowEntries = kColBlocksMax * 16 * 64;  // a row that takes a whole wave
//   A narrow layer (at most kNarrowUnits units) has a second form, for which the waves need no tables and whose next pieces
// they fetch four ahead: units of 64 lanes x 16 bytes.  A lane's first word: LDS slot of its row (kUnitIdleSlot: none), log2 of the
// lanes that its row takes (kUnitLanes, up to 64), kUnitRow if the row is flagged (see above); the others are kUnitEntries entries, dealt
// to the lanes of a row in turn.  Rows of several lanes come first, then those of more than three entries, then the others; a unit
// without rows of more than three entries a lane says so in its first lane (kUnitShort), whose row takes as many lanes as any
// of the unit.  What the streams add, in every lane: kUnitNew (the first unit of a layer), kUnitOr (of an OR layer), kUnitIdle (no
// rows), kUnitEnd (the wave has no further rows).
struct ColPlan {
    int32_t block_at[kColWaves + 1] = {}, table_at[kColWaves + 1] = {};   // first block / table of each wave
    std::vector<uint32_t> blocks, tables;
    int64_t share = 0;               // bound on the cost of a wave's share (cycles)
    std::vector<uint32_t> units;     // empty: the layer is none of the narrow ones
};
constexpr int kUnitEntries = 6, kUnitWords = 256, kUnitIdleSlot = 2, kUnitsAhead = 4;
constexpr uint32_t kUnitSlot = 0x7FFFu, kUnitRow = 1u << 18, kUnitShort = 1u << 19, kUnitNew = 1u << 20, kUnitOr = 1u << 21, kUnitIdle = 1u << 22,
                   kUnitEnd = 1u << 23;
constexpr int kUnitLanesAt = 15;     // three bits
constexpr int kNarrowUnits = 60;     // (30, 60 and 90 measured, see ColUnits)

// One gather-reduce pass set over a CSR whose rows are the outputs.
//   rows [0, n_main)                 write output row i; a split row holds the single entry kSkip
//   rows [n_main, n_main + n_seg)    are segments of split rows, writing scratch row (i - n_main)
//   combine: output row comb_row[h] reduces scratch rows comb_idx[comb_ptr[h] .. comb_ptr[h+1])
// Index entries carry the source row in bits 0..28, "last edge of its row" in bit 31, in the
// reverse sweep "weighted edge" in bit 30 (the parent is an OR node with more than one child), and on
// the last entry of a row bit 29 may flag the output row itself (reverse sweep into an OR layer: the row
// is an OR node with more than one child, whose adjoint is stored in the one-gather form).
// tasks: runs of consecutive main rows with a bounded edge count, as (first row, first edge)
// pairs with a closing (n_main, main edge count) pair: the unit of work of a wave of the edge kernel (the streaming
// kernel's: stream_tasks).
constexpr uint32_t kLastEdge = 0x80000000u, kWeightedEdge = 0x40000000u, kRowFlag = 0x20000000u, kSkipRow = 0xFFFFFFFFu;
// In the fused plans (LayerPlan::fwd2) that bit means something else: kGroupEnd on the last entry of a group.  The
// entries of a group are combined by the AND operation, the group results are the children of the OR row.
constexpr uint32_t kGroupEnd = kWeightedEdge;
// The OR rows that read through fused AND rows have at most this many entries (and at most half of
// Options::heavy_fan), so they are never split.  (Measured with 48 and the split threshold to match: 95% instead
// of 75% of the AND rows of the layered circuits fused, and the forward pass 3% slower: the long rows cost the
// fused launches more than the shorter AND launches save.)
constexpr int64_t kFusedRowMax = 24;
// Layers that a TopPlan may take have fused rows from this many nodes on, if one in this many is fused.
constexpr int64_t kTopFusedRows = 5000, kTopFusedShare = 4;
constexpr int64_t kMaxRows = (int64_t)1 << 29;      // row ids fit the 29-bit source field
constexpr int kIdxPad = 16;
// Split rows of more partial rows than this take a workgroup each in the combine pass, the others a wave.
constexpr int32_t kCombineWave = 16;

struct PassPlan {
    int32_t n_main = 0;
    int32_t n_seg = 0;
    int32_t n_heavy = 0;
    int32_t n_comb_many = 0;         // split rows of more than kCombineWave partial rows, the first ones of the combine lists
    int64_t edges = 0;
    std::vector<int32_t> ptr;        // [n_main + n_seg + 1]
    std::vector<uint32_t> idx;       // entries of all rows, zero padded by kIdxPad for chunked reads
    std::vector<int32_t> tasks;      // [2 * (n_tasks + 1)]
    int32_t n_tasks = 0;
    std::vector<int32_t> seg_tasks;  // same for the segment rows n_main .. n_main + n_seg - 1
    int32_t n_seg_tasks = 0;
    bool has_weighted = false;       // some entry carries kWeightedEdge
    std::vector<int32_t> seg_owner;  // [n_seg] output row each segment belongs to
    std::vector<int32_t> comb_ptr;   // [n_heavy + 1]
    std::vector<uint32_t> comb_idx;  // [n_seg + kIdxPad] scratch rows per split row, zero padded
    std::vector<int32_t> comb_row;   // [n_heavy]
};

struct LayerPlan {
    int64_t n = 0;                   // nodes in this layer
    int64_t e = 0;                   // edges from this layer down to layer - 1
    std::vector<int32_t> row_ptr;    // [n + 1] plain CSR by parent (Alg. 3: R_l implicit)
    std::vector<int32_t> child;      // [e]    S_l: position of the child in layer - 1
    std::vector<int32_t> origin;     // [n] input node id the row stands for
    std::vector<uint8_t> is_pad;     // [n] 1 for unary chain nodes
    std::vector<uint32_t> multi;     // [(n + 31) / 32] bit i: row i has more than one child (OR layers: the rows
                                     // whose edges carry a softmax weight in the reverse sweep)
    bool tail_ok = false;            // the layer may run in the persistent kernels
    // for those, in the layers tail_first .. num_layers: rows = nodes of this layer, sources = positions in layer - 1; rows =
    // nodes of layer - 1, sources = parents in this layer
    ColPlan col_fwd, col_bwd;
    PassPlan fwd;                    // outputs = nodes of this layer, sources = layer - 1
    PassPlan bwd;                    // outputs = nodes of layer - 1, sources = this layer
    // Fused AND rows (padding-free part only).  An AND node below layer alias_top that has at most one child
    // which is not a leaf and only OR parents whose rows stay short when they read its children instead of
    // it, is "fused": the forward plans below never read its value, so a forward sweep that uses them does not
    // have to write it.
    int64_t n_fused = 0;             // AND layers: so many of the rows are fused
    PassPlan fwd_kept;               // AND layers with fused rows: fwd with those rows left out (kSkipRow entries; launches have it without them, compact_pass)
    PassPlan fwd2;                   // OR layers that read fused rows: every child is a group of entries (kGroupEnd),
                                     // a fused AND child being replaced by its own children
};

// The narrow top of a circuit with long rows (power-law fan-ins), for the persistent kernels.  The layers of the circuit
// plan itself stay padding-free there (a chain node would cost the ordinary launches a row for each layer it passes); this plan
// holds the same nodes with the chain nodes that the kernels need, which exist only in their LDS.
//   Level l holds the nodes of layer l and a stand-in for every lower node that is read from above l.  Its first `kept` rows are
// those that the reverse sweep visits and whose values the forward kernel keeps; the rest are, at levels below alias_top, the
// stand-ins of nodes below the plan, whose adjoints the launches below gather from the rows of their parents.
struct TopPlan {
    struct Level {
        int64_t n = 0, kept = 0, e = 0;      // rows, rows kept, edges down to the level below
        int64_t at = 0;                      // first entry in a column of the value buffer
        int32_t launches = 0;                // kernel launches that the layer takes otherwise
        std::vector<int32_t> own;            // activation row of the node a row stands for
        ColPlan fwd, bwd;                    // bwd: the step into the level below (kept rows of both); empty at `first` unless that is 1
    };
    int32_t first = 0;                       // lowest layer it can take (0: there is no such plan)
    std::vector<Level> levels;               // first - 1 .. num_layers
    int64_t rows = 0;                        // kept rows of the levels first .. num_layers
    std::vector<int32_t> act_row;            // [rows] the activation row whose value and adjoint a kept row is, or -1 (stand-ins that have none)
    std::vector<uint32_t> multi;             // as LayerPlan::multi, rows of the top level
    std::vector<int32_t> root_pos, top_ptr, top_root;    // as in CircuitPlan, positions in the top level
    const Level& level(int32_t l) const { return levels[(size_t)(l - first + 1)]; }
    Level& level(int32_t l) { return levels[(size_t)(l - first + 1)]; }
};

struct CircuitPlan {
    int32_t num_vars = 0, num_roots = 0, num_layers = 0;
    std::vector<LayerPlan> layers;       // 0 .. num_layers
    std::vector<int32_t> leaf_code;      // layer 0: +(v+1), -(v+1), INT32_MAX (TRUE), INT32_MIN (FALSE)
    std::vector<int32_t> pos_row, neg_row;   // [V] layer-0 row of each literal or -1
    std::vector<int32_t> root_pos;       // [R] position of each root in the top layer
    std::vector<int32_t> top_ptr, top_root;  // top-layer node -> root columns that read it
    int64_t num_nodes = 0, num_edges = 0, dag_nodes = 0, dag_edges = 0, num_pad_nodes = 0;
    int64_t max_layer_nodes = 0, max_fan_in = 0, max_fan_out = 0, num_split_rows = 0;
    int64_t num_merged = 0;              // input gates identified with an identical gate
    int64_t max_fwd_seg = 0, max_bwd_seg = 0;   // scratch rows needed by split passes
    int32_t tail_first = 0;              // layers tail_first..num_layers may run in the persistent kernels (0: none)
    // Column-major value buffer of the persistent kernels: first entry of each layer in a column (-1: none).  The
    // layers tail_first .. num_layers follow one another from 0, the layer below tail_first comes after them.
    std::vector<int64_t> col_off;
    int64_t col_rows = 0;                // entries of the layers tail_first .. num_layers
    // Padding-free lower part (Options::alias_chains): layers 1 .. alias_top hold no chain nodes, except
    // that layer alias_top holds a stand-in for every node read from above it.  Their child entries are
    // rows of the whole activation buffer (row0[l] = first row of layer l), and layers[l].bwd for
    // l <= alias_top gathers the adjoints of layer l-1 from parents in any layer up to alias_top (adjoint
    // rows numbered like activation rows).  Layers above alias_top are as in the paper: child entries and
    // reverse-sweep sources are positions in the neighbouring layer.  0: the paper's layerization
    // throughout; num_layers: no chain nodes except the stand-ins of roots in the top layer.
    int32_t alias_top = 0;
    bool alias = false;                  // alias_top > 0
    int64_t num_fused = 0;               // AND rows whose values the fused plans do not need
    std::vector<int64_t> row0;
    TopPlan top;
};

// Status codes mirror klay_status (0 ok, 1 invalid, 2 cycle, 3 no memory).
int layerize(int32_t num_vars, int64_t num_nodes, const uint8_t* node_type, const int32_t* node_lit,
             const int64_t* child_ptr, const int32_t* child_idx, int32_t num_roots,
             const int32_t* roots, const Options& opt, CircuitPlan& plan, std::string& err);

// Split a CSR (n rows, ptr[n+1], idx) into main rows, segments and combine rows.
// `flags` (optional, one per edge) is OR-ed into the entries.
// `row_bits` (optional, a bit per output row) puts kRowFlag on the last entry of the flagged rows (for a
// split row: on the last entry of its combine list).
// `skip` (optional, a byte per row): rows to leave out; like a split row such a row is one kSkipRow entry.
void make_pass_plan(int64_t n, const int32_t* ptr, const int32_t* idx, const Options& opt, PassPlan& out,
                    const uint32_t* flags = nullptr, const uint32_t* row_bits = nullptr, const uint8_t* skip = nullptr);

// A plan without the main rows that it leaves out (kSkipRow entries), for launches: `out` numbers the others from 0 on (segments after
// them, as in any plan; the combine rows keep their numbers; no tasks of the edge kernel), out_row[i] is the row that row i of `out` writes,
// entry_row[j] the one that main entry j belongs to (padded like the entries).
void compact_pass(const PassPlan& in, PassPlan& out, std::vector<int32_t>& out_row, std::vector<int32_t>& entry_row);

// Tasks of the streaming kernel over the rows from .. to of a plan: (first row, its first entry, end of the rows, of the entries) of
// runs of rows with a bounded number of entries and without kSkipRow entries, and in the same kTaskWords words the first entries (as
// idx has them from there on): a wave that has its task can gather.
constexpr int kTaskWords = 16, kTaskHead = 4;
std::vector<int32_t> stream_tasks(const PassPlan& p, int64_t from, int64_t to);
// Entries that a wave reads of a task, from the first one on: the chunk in hand and two more, which it asks for before it knows whether
// the task has them.
constexpr int kStreamChunk = 4;
constexpr int64_t stream_reads(int64_t entries) { return (entries + kStreamChunk - 1) / kStreamChunk * kStreamChunk + 2 * kStreamChunk; }
// Where it reads as many output rows of them, in a plan of compact_pass.  The rows of a segment are not looked up, and entry_row ends with
// the main entries: a wave that has one reads the entries themselves in their place, without a branch.
constexpr const void* task_entry_rows(const uint32_t* idx, const int32_t* entry_row, int32_t first, bool segment) {
    return segment ? static_cast<const void*>(idx + first) : entry_row + first;
}

// Runs (see ColPlan) of a CSR of n rows for `waves` waves.  pad: slot that padding names; step: whose costs to
// cut by.  flags and row_bits as for make_pass_plan.
// The units of a narrow layer are part of it.
enum ColStep { kColFwdAnd, kColFwdOr, kColBwdAnd, kColBwdOr };
void make_cols(int64_t n, const int32_t* ptr, const int32_t* idx, const uint32_t* flags, const uint32_t* row_bits,
               int waves, int pad, ColStep step, ColPlan& out);
// The units of a layer (see ColPlan), none if they are more than `most`.
void make_units(int64_t n, const int32_t* ptr, const int32_t* idx, const uint32_t* flags, const uint32_t* row_bits, int pad, int most,
                std::vector<uint32_t>& units);

}  // namespace klay
