// Launch planning of the projection kernels: plain host arithmetic, no HIP types, so that it can be
// compiled and checked on a machine without a GPU.
#ifndef SS_PLAN_H
#define SS_PLAN_H

#include <cstddef>
#include <vector>

namespace ss {

// EPI_RESIDUAL and EPI_QKV: block kernel without k-slices only.  A plan for them is one for EPI_PARTIAL that, in the block kernel, counts what
// finishing costs with and without k-slices.
enum Epilogue { EPI_PARTIAL = 0, EPI_SWIGLU = 1, EPI_RESIDUAL = 2, EPI_QKV = 3 };

constexpr int kSweepMaxRows = 192;   // 12 row strips: beyond, the sweep kernel is never the faster one (see sweep_rows)

constexpr int kNarrowMaxRows = 96;   // most token-rows for which the 12-bit weights are read

// 16-byte units from one strip of a 12-bit matrix to the next: 3 KiB for each group of 4 k-blocks, and a gap.  The units of the
// chip stream different strips at about the same k, and where strips begin at multiples of 32 KiB, or are long, their requests
// meet in the same parts of the memory: a gap of 4 KiB, of 12 above 240 KiB where it is no multiple of 32, sends them to different ones.  Whole decode step, without gaps /
// with them: 7B widths, 12 layers (strips of 96 and 258 KiB) one row 0.955 / 0.888 ms, 16 rows 0.994 / 0.930, 64 rows 1.286 / 1.274, 96 rows
// 1.539 / 1.542; 8192 wide, 4 layers (192, 516 KiB) 0.954 / 0.883, 0.980 / 0.911, 1.184 / 1.142, 1.436 / 1.424; 13B widths (120, 324 KiB), 2048,
// 2816, 3072 and 6144 wide within 0.5 % either way.  Other gaps: 6 KiB instead of 12 for the long ones 7B 96 rows 1.550; at strips of 120 and 144
// KiB one row the same, 16 rows up to 4 % slower with 6.
constexpr size_t narrow_strip(int k_blocks)
{
    const int kib = k_blocks / 4 * 3;
    return (size_t)(kib + (kib % 32 == 0 ? 4 : kib > 240 ? 12 : 0)) * 64;
}

// Block kernel: tiles in 16-row strips, workgroups that share a compute unit, and the time of one k-block in
// nanoseconds while a unit holds one workgroup and while it holds per_cu of them; few: the part of trip_one that is left
// when next to no unit is busy (the others' power is theirs).
struct BlockTile {
    int ms, ns, per_cu;
    double trip_one, trip_full, few;
};
constexpr int kBlockTiles = 15;
extern const BlockTile block_tiles[kBlockTiles];

// Block kernel: the tile of workgroup b.  Workgroup ids are dealt to the 8 dies round-robin; the tiles a die works on at one time share
// their operands through its L2.  Few row tiles: panels of 8 of them, column tile by column tile inside a panel, a contiguous share for
// each die.  Many (4 or more for each die): a die keeps its own row tiles and takes them through all columns, so that the dies read
// the same weights at about the same time, once from HBM (fetching a line from afar is also power, which the matrix cores then lack:
// gate|up, 12311 rows, 1628 -> 1603 us); what is left over goes in panels as above.
constexpr int kBlockOwnFrom = 4, kBlockOwnStrips = 16;   // row tiles per die, and strips of a tile, from which a die keeps its own
struct BlockPlace {
    int n_tile, m_tile;
};
constexpr BlockPlace block_place(int b, int n_ntiles, int n_mtiles, int tile_strips)
{
    const int x = b & 7, own = tile_strips >= kBlockOwnStrips && n_mtiles >= 8 * kBlockOwnFrom ? n_mtiles >> 3 : 0, i = (b >> 3) - own * n_ntiles;
    if (i < 0) return {(b >> 3) / (own > 1 ? own : 1), x * own + (b >> 3) % (own > 1 ? own : 1)};
    const int rest = n_ntiles * n_mtiles - 8 * own * n_ntiles, per = rest >> 3, extra = rest & 7;
    const int t = x * per + (x < extra ? x : extra) + i;
    const int panel = t / (8 * n_ntiles), in_panel = t % (8 * n_ntiles), left = n_mtiles - 8 * own - panel * 8, ph = left < 8 ? left : 8;
    return {in_panel / ph, 8 * own + panel * 8 + in_panel % ph};
}

struct GemmPlan {
    int ksplit, nb, kd;
    int sweep_p, sweep_gn;
    int sweep_kh;   // sweep kernel: waves per unit (1 or 2)
    int narrow;     // sweep and skinny kernels: > 0 if the 12-bit form of the weights is read where the matrix has one;
                    // sweep kernel: then this many waves per unit
    int block;      // block kernel: index into block_tiles; -1: one of the others
};

// Few rows (k_gemm_few): how a workgroup of kFewWaves waves computes the sums that the sweep or skinny kernel would, in the same chains.
// A wave takes an item of a unit: the k-blocks of a slice (kb_slice), or one of `parts` parts of it: 2 parts take its groups of 4
// k-blocks in turn (sweep kernel, two waves per unit), 4 parts a quarter each (skinny kernel).  wave_kb: the slice's quarters are chains of
// their own also where one wave takes them all.  items: those of a unit; units_wg: units of a workgroup (0: no such plan).
// kFewRows: where the two meet on the wider matrices; ms per step of 12 layers of the 7B widths, others / these kernels: 4 rows 0.897 / 0.871,
// 5 rows 0.898 / 0.900, 6 rows 0.901 / 0.920; 13B widths, 8 layers, 5 rows 0.856 / 0.840; 2048 wide, 5 rows 0.517 / 0.483, 6 rows 0.516 / 0.497.
constexpr int kFewRows = 4, kFewWaves = 8, kFewMaxK = 16384;
struct FewPlan {
    int units_wg, items, parts, kb_slice, wave_kb;
};
FewPlan few_plan(int N, int Kp, int n_rows, int epilogue, int n_cu, int max_ksplit = 8);
// Its LDS: the rows, 64 bytes apart, the waves' sums, the rows' sums of squares.
constexpr size_t few_lds_bytes(int rows, int Kp, int epilogue)
{
    return (size_t)rows * (Kp + 32) * 2 + (size_t)kFewWaves * (epilogue == EPI_SWIGLU ? 2 : 1) * 1024 + (size_t)rows * 64;
}

// Token-rows (in whole strips) from which the block kernel may use its tile of 256 x 256: from the first that is priced by its products.  Below,
// two of them at most share a column of weights, and smaller tiles spread those over more units.  Barred up to 880 rows, as it was when there were five
// tiles: 494 rows, gate|up of 13B 137.8 us instead of 115.0, 6144 wide 170.7 / 150.8, 4096 wide with an MLP of 14336 110.4 / 96.0.
constexpr int kBlockTallFrom = 272;

// n_cu: compute units of the device (the sweep kernel runs one workgroup per unit).
// max_ksplit: 1 when the consumer reads the output directly (logits).
GemmPlan gemm_plan(int N, int Kp, int m_rows, int epilogue, int n_cu, int max_ksplit = 8);

// Strips per wave of the sweep kernel for this epilogue and row count.
int sweep_nbw(int epilogue, int m_rows);

// Rows a [ksplit][rows][N] partial-sum buffer must hold so that every plan gemm_plan can return for an
// [N, *] matrix and 1 <= m_rows <= n_max fits: an upper bound of ksplit * m_rows over that range.
size_t gemm_partial_rows_bound(int n_max);

// Rows up to which the sweep kernel is chosen for a matrix of w_per_cu weight bytes per compute unit and this many units.
int sweep_rows(size_t w_per_cu, int units, int n_cu);

// Decode steps of small models: whether n_rows rows with contexts of at most max_ctx slots go through k_row_step, one
// workgroup for a row's whole step, instead of 7 launches per layer.
constexpr int kRowMaxLayers = 16;
constexpr int kRowWaves = 8;
constexpr int kRowMaxModel = 64 * kRowWaves;   // model width: a thread per element, and at least a wave per head
constexpr int kRowMaxFfn = 8192;
bool row_step_plan(int n_layers, int d, int F, int V, int n_rows, int max_ctx, int n_cu, int hd = 64);
constexpr int row_padded(int k) { return (k + 255) / 256 * 256; }   // whole groups of 8 k-blocks
// Its LDS: residual row, query, rotation, attention sums of every wave, the two projection inputs, this position's key and value.
constexpr size_t row_step_lds_bytes(int d, int Fp, int hd)
{
    return (size_t)(2 * d + hd + kRowWaves * (hd + 4)) * 4 + (size_t)(row_padded(d) + row_padded(Fp) + 2 * d) * 2;
}

// Decode attention: (row, head) pairs of a whole micro-batch up to which 16 waves each are used, once some context exceeds
// what 8 have in flight.
constexpr int kAttnWidestMaxGroups = 192;
constexpr bool attention_may_widen(int mb_rows, int H, int max_ctx, int hd)
{
    return mb_rows * H <= kAttnWidestMaxGroups && max_ctx > 64 * (512 / hd);
}

constexpr int kWorkspaceRows = 128;   // activation buffers hold whole multiples of this many token-rows

// Workgroups that share out the slots of one pair (1: no split), up to kAttnMaxSplit, at least kAttnSplitSlots slots each, and so
// few that their sums fit a buffer of kWorkspaceRows rows.
constexpr int kAttnMaxSplit = 16, kAttnSplitSlots = 256, kAttnSplitMaxGroups = 96;
int attention_split(int mb_rows, int H, int hd, int max_ctx);
// Floats that the shares of n_rows rows take: the sums of a head, their maximum and their total each.
constexpr size_t attention_share_floats(int n_rows, int H, int hd, int split) { return (size_t)n_rows * H * split * (hd + 2); }

// ... and 8 waves each (else 4).  The slots are dealt to 8 slices, whatever the waves, for every row count of a strip that holds
// one so small: a row's numbers are not to depend on who else is still alive, its time may.  (40 heads, 16 rows that become
// fewer; 4 slices for the whole strip / 8, decode step of 13B per layer, us: 16 rows at context 50 110.6 / 111.0, 3 rows at 300 113.4 / 111.4,
// one row at 600 117.5 / 113.7; without the MLP 4 rows at 3000 141.6 / 118.6.)
constexpr int kAttnWideMaxGroups = 512;
constexpr bool attention_wide(int n_rows, int H) { return n_rows * H <= kAttnWideMaxGroups; }
constexpr int attention_fewest_rows(int n_rows) { return (n_rows + 15) / 16 * 16 - 15; }   // of n_rows' strip

// Launch shape of the decode attention: slices that a pair's slots are dealt to (their number is the order of the sums), waves
// that take them, workgroups that share out the slots.  n_rows: rows of the launch; plan_rows: rows that its sums are planned for
// (n_rows, or those of one micro-batch of several); mb_rows: rows of the micro-batch, finished ones included; max_ctx: longest
// context in this forward, were all alive.
struct AttentionPlan {
    int slices, waves, split;
};
AttentionPlan attention_plan(int n_rows, int plan_rows, int mb_rows, int H, int hd, int max_ctx);

// Micro-batches of a group pass that share their decode forwards: rows of one (a strip: every plan of a strip holds for it
// alone and for several together) and of all.
constexpr int kSharedMbRows = 16, kSharedRows = 64;
// One of them: its longest prompt, and forwards, counting the prompt's.  The longest context of forward g is that of the
// micro-batches that still take part: each stays below where its attention would widen, and so do those that are there.
struct SharedShape {
    int prompt, steps;
};
int shared_context(const SharedShape* mb, int n_mb, int g);
// Whether they do: where a launch is the time of its weights (7 MB and more each, 7 a layer).  Below that it is the time of
// a launch, which several streams hide better.  Group passes, four micro-batches in flight on streams / sharing, ms: 4 layers
// 512 wide 22.4 / 27.3, 12 layers 1024 wide (25 MB a layer) 74.5 / 85.4, 6 layers 2048 wide (101 MB) 63.6 / 61.8 and 31.7 / 26.3,
// 4 layers 3072 wide 69.9 / 54.6, 4 layers of 7B 121 / 82 and 64 / 35.
constexpr bool shared_forwards_pay(int d, int F) { return ((size_t)4 * d * d + (size_t)3 * d * F) * 2 >= (size_t)50 << 20; }

// How a group pass hands out its micro-batches, given in the order of their length: those that share their decode forwards, as many
// as may be in flight, or one fewer if others are there to run beside them; and those that run one at a time, the left-over that
// found no company among them.  beside[u]: lanes that may run while shared unit u and those after it do.
struct PassUnits {
    std::vector<std::vector<int>> shared, alone;
    std::vector<int> beside;
};
PassUnits pass_units(const std::vector<int>& order, const std::vector<int>& rows, const std::vector<char>& can_share, int lanes);

// Testing aid: 0 = choose per shape (default), 1 = never use the sweep kernel, 2 = use it for every
// projection of at most kSweepMaxRows rows.
void set_gemm_mode(int mode);
int gemm_mode();

}  // namespace ss

#endif
