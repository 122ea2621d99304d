// Which kernel runs a projection, and in which launch shape (host arithmetic only).
#include "ss_plan.h"

#include <algorithm>
#include <atomic>
#include <cmath>

namespace ss {

namespace {
std::atomic<int> g_gemm_mode{0};
std::atomic<int> g_sweep_split{1};
std::atomic<int> g_tall_tiles{1};
std::atomic<int> g_block_tile{-1};
constexpr int kSmallMaxKsplit = 8;   // sweep and skinny kernels: at most 8 k-slices
// Block kernel: rows up to which k may be cut in 4 and in 2 (more rows fill the chip without, and the partial sums of
// every slice are written and read again)
constexpr int kBlockRows4 = 512, kBlockRows2 = 2048;
// ns for launch, first stage and epilogue; bytes per ns at which results are written and at which the weights arrive at best
struct BlockRates {
    double start, write, stream;
};
constexpr BlockRates kBlockRates = {4390.0, 9.59, 3.3};
constexpr double kPartialRead = 4.5;          // bytes per ns at which the consumer adds further slices
constexpr double kRotateStart = 3000.0;       // ns of the launch that rotates slices of q|k|v
// Tiles of which a unit holds two, from so many full rounds and up to so many k-blocks on: the workgroups of a unit have drifted apart, and one
// multiplies while the other starts or finishes (gate|up, 12311 rows, tiles of 192 x 192 / 384 x 192: 1560 / 1607 us; down, 344 k-blocks: 937 / 871).
// Where between 192 and 344 k-blocks the line lies made no difference (8192 wide; MLPs of 6912 and 8192).
constexpr int kBlockManyRounds = 4, kBlockManyTrips = 192;
constexpr double kBlockManyGain = 0.987;
constexpr double kBlockPad = 0.08;             // share of the products beyond the matrix that is paid for again, in power
constexpr double kBlockHalfPair = 0.593;      // of trip_full, when next to no unit holds a second workgroup
// Large matrices, up to so many rows: the weights' way from memory decides more than the products, idle units make nothing faster, and
// only the first five tiles, with rates of their own (trip_one and trip_full), are chosen from: of those there, smaller ones were
// faster only where the weights came from the memory-side cache.
constexpr int kBlockStreamRows = 256, kBlockStreamTiles = 5;
constexpr BlockRates kBlockStreamRates = {3300.0, 3.84, 3.64};
constexpr double kBlockStreamTrips[kBlockStreamTiles][2] = {{615.0, 740.0}, {485.0, 613.0}, {412.0, 772.0}, {313.0, 619.0}, {239.0, 475.0}};
// Weights up to here stay in the L2s of the dies from forward to forward; tiles of fewer than 64 blocks of 16 x 16, which fetch the most
// bytes per product, are for them (measured up to kBlockRows2 rows).
constexpr size_t kBlockCached = (size_t)16 << 20;

}

// Fitted to 3000 timings inside prompt forwards of the 7B and 13B shapes, 304 to 12311 rows, every tile in turn (a projection that is launched
// over and over finds its weights and its clock otherwise than one between others: up to 18 % apart, and not the same for all tiles), and to 1500
// of launches alone at widths of 256 and 2048.  With more sizes to choose from tiles fill whole rounds of the 256 units.  Timed anew inside forwards, every
// tile in turn, how much slower than the best one are the tile taken / the best of the first five, which were all there was: 88 projections of the
// 7B and 13B shapes 0.8 / 4.1 %; 336 of nine shapes from 1280 to 8192 wide that those forwards did not hold 1.2 / 4.5 % (27 % at worst); 240 of matrices up to 16 MB,
// 640 to 2048 wide, 1.1 / 12.5 %.  Against the choice among five, 32 of the 664 are 2 to 12 % slower, none of 7B and 13B, and all together 8 % faster.
// The last digits are those with which the choice is best.  Fitted to launches alone, without what a launch's last step costs (finish_bytes), the tile
// taken was 3.1 % slower at 7B and 13B.  Microseconds in a forward, with the consumer's reads, that fit / this one: 7B o 995 rows 44 / 39, 2033 rows 75 / 69, down 995 rows
// 89 / 86, gate|up 7200 rows 976 / 936, 12311 rows 1607 / 1560; 13B o 608 rows 53 / 43, 995 rows 70 / 57, down 12311 rows 1350 / 1304.
const BlockTile block_tiles[kBlockTiles] = {
    {16, 16, 1, 704.0, 736.0, 1.0}, {16, 12, 1, 554.0, 590.0, 0.91}, {8, 16, 2, 449.0, 773.0, 0.79}, {8, 12, 2, 346.0, 638.0, 0.71},
    {8, 8, 2, 261.0, 493.0, 0.55}, {8, 4, 2, 155.0, 404.0, 0.89}, {6, 8, 2, 223.0, 549.0, 0.98}, {10, 8, 2, 296.0, 576.0, 0.66},
    {12, 8, 2, 321.0, 635.0, 0.74}, {16, 8, 1, 389.0, 425.0, 0.86}, {10, 12, 2, 424.0, 756.0, 0.75}, {12, 12, 2, 446.0, 824.0, 0.89},
    {14, 16, 1, 594.0, 670.0, 1.0}, {20, 12, 1, 624.0, 700.0, 1.0}, {24, 12, 1, 743.0, 823.0, 1.0}};

namespace {
bool cached(int N, int Kp) { return (size_t)N * Kp * 2 <= kBlockCached; }
bool stream_bound(int N, int Kp, int m_rows) { return m_rows <= kBlockStreamRows && !cached(N, Kp); }

// What an unsliced launch's results cost, as bytes written per element: the rows of the residual stream are read first, and every
// workgroup waits for its own at the end; rotated elements go to three places.
double finish_bytes(int epilogue) { return epilogue == EPI_RESIDUAL ? 16.4 : epilogue == EPI_QKV ? 6.0 : 4.0; }

// Time of a projection in the block kernel, in nanoseconds: rounds of workgroups over the chip times the k-blocks of a
// slice, the results, and what adding up the slices costs the consumer.
double block_ns(const BlockTile& t, int ks, int N, int Kp, int m_rows, int epilogue, int n_cu)
{
    const long long strips_m = (m_rows + 15) / 16, strips_n = N / 16;
    const long long wgs = ((strips_m + t.ms - 1) / t.ms) * ((strips_n + t.ns - 1) / t.ns) * ks;
    const long long full = wgs / ((long long)n_cu * t.per_cu), rest = wgs % ((long long)n_cu * t.per_cu);
    const double busy = (double)rest / n_cu;
    const int trips = (Kp / 32 + ks - 1) / ks;
    BlockRates r = kBlockRates;
    double trip, bytes = epilogue == EPI_SWIGLU ? 1.0 : 4.0 * ks;
    const bool large = !cached(N, Kp) && m_rows > kBlockStreamRows;
    if (stream_bound(N, Kp, m_rows) && &t - block_tiles < kBlockStreamTiles) {
        const double* ns = kBlockStreamTrips[&t - block_tiles];
        r = kBlockStreamRates;
        trip = (double)full * ns[1] + (rest > n_cu ? ns[1] : rest > 0 ? ns[0] : 0.0);
    } else {
        const double last = rest > n_cu ? t.trip_full * (kBlockHalfPair + (1.0 - kBlockHalfPair) * busy / t.per_cu)
                                        : rest > 0 ? t.trip_one * (t.few + (1.0 - t.few) * busy) : 0.0;
        // small tiles run behind their weights in long loops (an exponent of 0.35, fitted to launches alone at widths of 256 and 2048, made short
        // loops too cheap: 1536 wide, 2033 rows, o 32 us with what follows instead of 26; 768 wide, 2033 rows, gate|up 27 instead of 21)
        trip = ((double)full * t.trip_full + last) * std::pow(trips / 128.0, t.ms * t.ns < 64 ? 0.1 : -0.108);
        if (t.per_cu == 2 && full >= kBlockManyRounds && trips <= kBlockManyTrips) trip *= kBlockManyGain;
        // tiles that reach past the matrix multiply there as well: units that would idle cost less of the chip's power
        if (large) trip *= 1.0 + kBlockPad * ((double)(wgs / ks) * t.ms * t.ns / ((double)strips_m * strips_n) - 1.0);
        if (large && ks == 1 && epilogue != EPI_SWIGLU) bytes = finish_bytes(epilogue);
    }
    const double cells = (double)m_rows * N;
    const double work = r.start + trip * trips + cells * bytes / (r.write * 1000.0);
    const double stream = r.start + (double)N * Kp * 2 / (r.stream * 1000.0);
    const double ns = work > stream ? work : stream;
    if (epilogue == EPI_SWIGLU || ks == 1) return ns;
    // sliced q|k|v of a prompt forward: a launch that rotates reads all slices
    if (epilogue == EPI_QKV && !stream_bound(N, Kp, m_rows)) return ns + kRotateStart + cells * 4.0 * ks / (kPartialRead * 1000.0);
    return ns + cells * 4.0 * (ks - 1) / (kPartialRead * 1000.0);
}
}

void set_gemm_mode(int mode)
{
    // bit 2 (value 4) added to a mode: the sweep kernel never splits a unit between two waves (A/B measurements)
    g_sweep_split.store((mode & 4) ? 0 : 1, std::memory_order_relaxed);
    // bit 3 (value 8): the block kernel never uses its tile of 256 x 256 (A/B measurements)
    g_tall_tiles.store((mode & 8) ? 0 : 1, std::memory_order_relaxed);
    // bits 4 and up: 1 + the only tile the block kernel uses
    g_block_tile.store((mode >> 4) - 1, std::memory_order_relaxed);
    g_gemm_mode.store(mode & 3, std::memory_order_relaxed);
}
int gemm_mode() { return g_gemm_mode.load(std::memory_order_relaxed); }

// Launch shape of a projection.
// Sweep kernel (up to sweep_rows rows, at least 160 KiB of weights per compute unit and row strip; below that the launch is
// too short to amortise its start-up and the skinny kernel's finer split wins: measured at 16 rows, the 7B o
// projection, 131 KiB per unit, is 12 % faster in the skinny kernel, the 13B one, 205 KiB, 30 % faster here): one workgroup per compute unit and
// k-slice, a wave per output strip (per gate/up strip pair with the SwiGLU epilogue).  k-slices double
// until every workgroup has 4 or more waves of work, as far as the epilogue allows them, never below 16
// k-blocks per slice; a workgroup has 4 or 8 waves, and when 8 are not enough there are more workgroups.
// Skinny kernel (<= 64 rows otherwise), from sweeps on the 7B shapes: aim at 512+ workgroups; 4 strips per
// workgroup halve the activation re-reads and win when k is short, 2 strips when k is long or when the
// epilogue forbids k-slices (SwiGLU, logits); k-slices double until there are 512 workgroups, at most 8,
// never leaving a wave fewer than 4 k-blocks.  Block kernel (everything else): the tile and the number of k-slices
// with the smallest estimated time.

// Strips per wave of the sweep kernel: a gate/up pair for the SwiGLU epilogue, otherwise one.  One strip per wave gives
// twice the units of two, so half the k-slices (longer sweeps, half the partial sums).  Two strips per wave halve the LDS
// operand reads per weight byte and were the better choice from 49 rows on while an activation was two operands; with
// one operand per activation they never are.  Same GPU, 7B shapes, decode step at context 100, one / two strips per wave:
// 64 rows 3.99 / 4.27 ms, 80 rows 4.36 / 4.58, 96 rows 4.82 / 5.04, 128 rows 5.59 / 5.81.
int sweep_nbw(int epilogue, int /*m_rows*/) { return epilogue == EPI_SWIGLU ? 2 : 1; }

// Rows up to which the sweep kernel is chosen before the block kernel (the sweep's cost grows with every strip, the block
// kernel computes whole tiles of 128 rows but streams nothing twice).  The more weights a compute unit has to stream, and
// the fewer k-slices it takes to occupy them all, the longer the sweep stays ahead.  Microseconds, sweep / block:
//   little weight   d 1024 gate|up 160 rows 13.1 / 11.3; d 2048 gate|up 160 rows 21.4 / 20.3; 7B o 160 rows 16.5 / 15.6
//   k in slices     13B o 160 rows 20.7 / 22.8; down 160 rows 45.3 / 47.7, 176 rows 51.1 / 48.2; 7B down 176 rows 34.1 / 32.9
//   neither         7B q|k|v 160 rows 32.7 / 34.8, 192 rows 35.8 / 35.2, gate|up 176 rows 54.0 / 56.8, 192 rows 56.4 / 58.5,
//                   208 rows 68.0 / 58.3, head 192 rows 78.5 / 85.6; 13B gate|up 192 rows 83.3 / 94.3; d 8192 139 / 157
int sweep_rows(size_t w_per_cu, int units, int n_cu)
{
    if (w_per_cu < ((size_t)192 << 10)) return 144;
    return units > 2 * n_cu && w_per_cu >= ((size_t)384 << 10) ? kSweepMaxRows : 160;
}

GemmPlan gemm_plan(int N, int Kp, int m_rows, int epilogue, int n_cu, int max_ksplit)
{
    GemmPlan p{1, 2, 4, 0, 0, 1, 0, -1};
    // whole strips: a micro-batch keeps its launch shapes, and its rows their last bits, while it shrinks inside a strip
    m_rows = (m_rows + 15) / 16 * 16;
    const int KB = Kp / 32;
    const int mode = gemm_mode();
    if (m_rows <= kSweepMaxRows) {
        const size_t w_per_cu = (size_t)N * (size_t)Kp * 2 / (size_t)n_cu;
        const size_t mt_rows = (size_t)(m_rows + 15) / 16;   // activation re-reads grow with the row strips: sweep earlier
        const int nbw = sweep_nbw(epilogue, m_rows);
        const int units = (N / 16 + nbw - 1) / nbw;
        if (mode == 2 ||
            (mode == 0 && m_rows <= sweep_rows(w_per_cu, units, n_cu) && w_per_cu * mt_rows >= ((size_t)160 << 10))) {
            if (epilogue == EPI_SWIGLU) max_ksplit = 1;   // fused epilogue: no k-slices
            while (units * p.ksplit < 4 * n_cu && p.ksplit * 2 <= max_ksplit && p.ksplit < kSmallMaxKsplit &&
                   KB / (p.ksplit * 2) >= 16)
                p.ksplit *= 2;
            int gn = std::max(1, std::min(units, n_cu / p.ksplit));
            if ((units + gn - 1) / gn > 8) gn = (units + 7) / 8;
            p.sweep_p = (units + gn - 1) / gn <= 4 ? 4 : 8;
            p.sweep_gn = gn;
            // above 96 rows a workgroup with at most 4 units runs 8 waves, two per unit: the work per weight byte
            // grows with the row strips and 4 waves (one per SIMD) stop keeping up with the weight stream (same GPU,
            // split / not split: 104 rows 5.09 / 5.18 ms per step, 112 rows 5.21 / 5.28, 128 rows 5.59 / 5.81; up to
            // 96 rows the two are equal to within 0.1 %)
            if (Kp % 128 == 0 && m_rows <= kNarrowMaxRows)
                p.narrow = (p.sweep_p == 4 && g_sweep_split.load(std::memory_order_relaxed)) ? 2 : 1;
            p.sweep_kh = (p.sweep_p == 4 && m_rows > 96 && g_sweep_split.load(std::memory_order_relaxed)) ? 2 : 1;
            return p;
        }
    }
    if (m_rows <= 64) {
        if (epilogue == EPI_SWIGLU) max_ksplit = 1;   // fused epilogue: no k-slices
        const int mt = (m_rows + 15) / 16;
        p.kd = mt == 1 ? 4 : 2;
        // the kernel reads 12-bit weights 4 k-blocks at a time, and its 4 waves take whole groups: below 16 k-blocks some
        // would have none (such matrices are small enough to stay in L2, where their bytes are not what takes time)
        p.narrow = Kp % 128 == 0 && mt == 1 && KB >= 16;
        if (max_ksplit == 1 && epilogue == EPI_SWIGLU) return p;
        p.nb = (mt == 1 && KB > 256) ? 2 : 4;   // with several row strips the activation re-reads dominate: 4 strips
        if (max_ksplit == 1 && mt == 1) p.nb = 2;
        const int groups = (N / 16 + p.nb - 1) / p.nb;
        while (groups * p.ksplit < 512 && p.ksplit * 2 <= max_ksplit && p.ksplit < kSmallMaxKsplit &&
               KB / (p.ksplit * 2 * 4) >= 4)
            p.ksplit *= 2;
        return p;
    }
    if (epilogue == EPI_SWIGLU) max_ksplit = 1;   // fused epilogue: no k-slices
    const bool tall = m_rows >= kBlockTallFrom && g_tall_tiles.load(std::memory_order_relaxed);
    const int most = m_rows <= kBlockRows4 ? 4 : m_rows <= kBlockRows2 ? 2 : 1;
    double best = 0.0;
    const int only = g_block_tile.load(std::memory_order_relaxed);
    const int tiles = stream_bound(N, Kp, m_rows) ? kBlockStreamTiles : kBlockTiles;
    for (int t = only >= 0 ? only : tall ? 0 : 1; t < (only >= 0 ? only + 1 : tiles); ++t) {
        if (only < 0 && (!cached(N, Kp) || m_rows > kBlockRows2) && block_tiles[t].ms * block_tiles[t].ns < 64) continue;
        for (int ks = 1; ks <= std::min(most, max_ksplit) && (ks == 1 || KB / ks >= 16); ks *= 2) {
            const double ns = block_ns(block_tiles[t], ks, N, Kp, m_rows, epilogue, n_cu);
            if (p.block < 0 || ns < best) {
                best = ns;
                p.block = t;
                p.ksplit = ks;
            }
        }
    }
    return p;
}

FewPlan few_plan(int N, int Kp, int n_rows, int epilogue, int n_cu, int max_ksplit)
{
    FewPlan f{0, 1, 1, 0, 0};
    if (gemm_mode() != 0 || !g_sweep_split.load(std::memory_order_relaxed) || n_rows > kFewRows || Kp > kFewMaxK || Kp % 128) return f;
    if (few_lds_bytes(n_rows, Kp, epilogue) > (size_t)160 << 10) return f;
    const GemmPlan p = gemm_plan(N, Kp, n_rows, epilogue == EPI_RESIDUAL ? (int)EPI_PARTIAL : epilogue, n_cu, max_ksplit);
    if (!p.narrow || p.block >= 0) return f;
    const int nbw = epilogue == EPI_SWIGLU ? 2 : 1, units = N / 16 / nbw;
    f.kb_slice = ((Kp / 32 + p.ksplit - 1) / p.ksplit + 3) & ~3;   // whole groups, as the launchers cut them
    if (p.sweep_gn > 0) {
        const int per = (units + p.sweep_gn - 1) / p.sweep_gn;
        f.parts = p.sweep_p == 4 && per <= 4 && p.narrow == 2 ? 2 : 1;
    } else {
        f.wave_kb = 1;
        f.parts = p.ksplit * 4 <= kFewWaves ? 4 : 1;
    }
    f.items = p.ksplit * f.parts;
    if (f.items > kFewWaves) return f;
    f.units_wg = std::min(kFewWaves / f.items, std::max(1, (units + n_cu - 1) / n_cu));
    return f;
}

// Both ways to take a decode step of a small model, in microseconds, fitted to 1510 timings of either on 200 models of 1 to 16
// layers, 64 to 512 wide, 1 to 250 rows, contexts of 8 to 1500 (row step 5 % off in the root mean square, launches 6 %).  The row step is taken up to 3 us
// behind: all steps of a row in one launch save it another 7 us each, and micro-batches in flight beside each other hold each
// other up less in one launch a step than in dozens.  Of those points, one step each, 31 are more than 2 % slower than the
// other way, the mean over all is 0.2 % above that of the better way.  Microseconds, launches / row step: tiny (2 layers, 256 wide, 3.6 MB)
// 16 rows at context 8 65.0 / 47.8, 200 68.4 / 59.4, 600 72.7 / 70.4, one row 61.0 / 46.8, 600 65.5 / 68.0, 100 rows 8 99 / 50; 1 layer 64
// wide, 6000 ids 35.0 / 40.5, 2000 ids 34.2 / 25.7; 4 layers 64 wide, ffn 2048 103 / 128.  Tiny, a group of 64, prompts of 200, four micro-batches in
// flight: 10.6 ms in launches, 7.8 in row steps.
constexpr double kRowStepBehind = 3.0;

// A workgroup of k_row_step reads the whole model and its row's slots by itself: every pair of strips in whole groups of 8
// k-blocks (past the end the last block again), 16 KB each at 120 GB/s; its phases wait for each other.  A head's slots go to
// kRowWaves / heads waves, so some of them may be without.
static double row_step_us(int n_layers, int d, int F, int V, int max_ctx, int hd)
{
    const double groups = row_padded(d) / 256;
    const auto pairs = [](int strips) { return (double)((strips + 1) / 2); };
    const double layer = (pairs(3 * d / 16) + pairs(d / 16) + pairs(F / 8)) * groups + pairs(d / 16) * (row_padded(F) / 256);
    const double heads = d / hd, busy = heads * (int)(kRowWaves / heads) / kRowWaves;
    return 8.0 + n_layers * (6.2 + 0.135 * layer + 0.0139 * max_ctx * d / 256 / busy) + 0.135 * pairs(V / 16) * groups;
}

// The launches of the other kernels: each the time of a launch with so many strips of rows, the weights, and what the slots add
// (never more than in the row step: a context that grows does not turn a micro-batch back to it).
static double step_launches_us(int n_layers, int d, int F, int V, int n_rows, int max_ctx)
{
    const int strips = (n_rows + 15) / 16;
    const double launch = strips > 4 ? 4.4 + 0.5 * d / 256 : 3.0 + 0.24 * strips;
    const double mb = (n_layers * (4.0 * d * d + 3.0 * d * F) + (double)V * d) * 2e-6;
    return (7 * n_layers + 4) * launch + 0.6 * mb +
           std::min(0.005 + 0.003 * (strips - 1), 0.0139) * n_layers * max_ctx * d / 256;
}

bool row_step_plan(int n_layers, int d, int F, int V, int n_rows, int max_ctx, int n_cu, int hd)
{
    // the testing aids choose among the projection kernels: they get those
    if (gemm_mode() != 0 || g_block_tile.load(std::memory_order_relaxed) >= 0 || !g_sweep_split.load(std::memory_order_relaxed) ||
        !g_tall_tiles.load(std::memory_order_relaxed))
        return false;
    if (n_layers > kRowMaxLayers || d > kRowMaxModel || F > kRowMaxFfn) return false;
    if ((n_rows + 15) / 16 * 16 > n_cu) return false;   // a unit each, by whole strips like the other plans
    return row_step_us(n_layers, d, F, V, max_ctx, hd) - kRowStepBehind <= step_launches_us(n_layers, d, F, V, n_rows, max_ctx);
}

// Few pairs leave most of the chip idle over a long context; more workgroups each, and a launch that joins them.  By the
// micro-batch and its progress, like the waves.  Decode step of 7B per layer, us, 16 waves a pair / split: one row at context 1000
// 90.4 / 89.2, 1400 94.7 / 88.7, 2000 99.8 / 89.5, 3900 118 / 94; two rows 1000 90.9 / 90.4, 2000 101 / 94, 3900 121 / 105; three 1000
// 92.0 / 92.3, 2000 103 / 100, 3900 124 / 117; four 1000 92.3 / 93.4, 2000 104 / 106; six 2000 113 / 122 (what a unit of 16 waves
// keeps in flight is enough there).  Other heads (8 layers, or 17 of up to 512 wide, whole step per layer):
//   heads of 128   8 x 1 row 1030 35.9 / 35.4, 2100 42.5 / 35.0; 8 x 12 1030 43.7 / 43.8, 2100 56.3 / 51.0; 4 x 24 1030 43.4 / 43.5, 1300
//                  46.7 / 44.4; 16 x 6 1030 48.7 / 48.7: as with 32 heads, from 1024 slots
//   heads of 64    (half the bytes a slot) 32 x 1 1030 38.1 / 38.8, 1300 39.3 / 38.9; 32 x 3 1030 39.5 / 41.4, 1300 43.0 / 43.5, 2100 49.4 / 47.2;
//                  16 x 4 1600 35.9 / 36.3, 2100 42.1 / 39.1; 8 x 6 1030 31.5 / 32.1, 1300 35.3 / 34.3; 4 x 12 1300 33.2 / 32.1: from 1280, and
//                  from 1792 where there are more than 48 pairs
// With fewer than 5 heads the shares of many rows would not fit the buffer: fewer then.
int attention_split(int mb_rows, int H, int hd, int max_ctx)
{
    const int pairs = mb_rows * H;
    const int from = hd >= 128 ? 1024 : pairs <= kAttnSplitMaxGroups / 2 ? 1280 : 1792;
    if (pairs > kAttnSplitMaxGroups || max_ctx < from) return 1;
    const int fit = (int)((size_t)kWorkspaceRows * H * hd / attention_share_floats(mb_rows, H, hd, 1));
    return std::max(1, std::min({kAttnMaxSplit, (512 + pairs - 1) / pairs, max_ctx / kAttnSplitSlots, fit}));
}

namespace {
// Waves that take the slices of a pair; any number gives the same sums.  8 while all pairs are resident with room to spare, 4
// beyond.  With somewhat more pairs than the chip's 256 units, or than two for each, and long contexts, the units that have a pair
// more decide, and those that have not are not to take the memory's time from them: half as many waves, from 650 slots of 128
// elements or 1300 of 64 (two for each: 1000 and 2000).  Decode step per layer, us, 32 heads of 128 unless it says otherwise:
//   8 waves / 4   9 rows, context 500 71.6 / 71.4, 900 82.8 / 82.3, 1500 108.8 / 104.3, 3000 155.3 / 143.0; 12 rows 300 66.8 / 67.3, 900 92.3 /
//                 89.9, 1500 112.8 / 110.3; 14 rows 1500 117.9 / 118.2, 3000 179.6 / 180.9; 8 rows 900 76.2 / 79.5, 1500 94.8 / 100.1; heads of 64,
//                 32 x 11 900 54.3 / 54.5, 1500 65.0 / 63.5; 16 x 18 900 45.4 / 47.7, 1500 59.5 / 59.2, 3000 82.4 / 79.8
//   4 waves / 2   17 rows 400 83.6 / 85.6, 1000 122.5 / 122.0, 1500 149.8 / 147.7, 3000 232.3 / 222.3; 20 rows 1500 158.1 / 156.3; 40 x 13 1500
//                 155.3 / 152.3, 3000 234.0 / 224.4; heads of 64, 32 x 17 700 60.2 / 63.5, 1500 81.9 / 83.4, 2200 100.7 / 101.0, 3000 123.8 / 122.0
int attention_waves(int pairs, int hd, int max_ctx)
{
    if (pairs > kAttnWideMaxGroups) return pairs <= 640 && max_ctx * hd > 1000 * 128 ? 2 : 4;
    return pairs > 256 && pairs <= 416 && max_ctx * hd > 650 * 128 ? 4 : 8;
}
}

AttentionPlan attention_plan(int n_rows, int plan_rows, int mb_rows, int H, int hd, int max_ctx)
{
    // measured at the 7B shape: 8 waves win at 16 rows (512 workgroups: 14.1 against 14.9 us per layer at context
    // 200), 4 waves win at 64 rows (2048 workgroups: 25.7 against 36.1 us at context 100)
    // 16 waves where 8 would need a second round trip (3 rows at context 2400: 47.5 -> 38 us); shorter contexts leave some
    // of them without a slot (tiny model, context 40: 6 us with 8 waves, 7.3 with 16).  Their sums add up in another order,
    // so the choice depends on the micro-batch and on how far it has come, not on how many of its rows are still alive: a
    // row's numbers are to be the same whether or when the others leave.
    const int split = attention_split(std::max(mb_rows, n_rows), H, hd, max_ctx);
    if (split > 1) return {8, 8, split};
    if (attention_may_widen(mb_rows, H, max_ctx, hd)) return {16, 16, 1};
    const int slices = attention_wide(attention_fewest_rows(plan_rows), H) ? 8 : 4;
    return {slices, std::min(slices, attention_waves(n_rows * H, hd, max_ctx)), 1};
}

int shared_context(const SharedShape* mb, int n_mb, int g)
{
    int ctx = 0;
    for (int k = 0; k < n_mb; ++k)
        if (mb[k].steps > g) ctx = std::max(ctx, mb[k].prompt + g);
    return ctx;
}

PassUnits pass_units(const std::vector<int>& order, const std::vector<int>& rows, const std::vector<char>& can_share, int lanes)
{
    int n_share = 0;
    for (int k : order) n_share += can_share[k];
    const int together = n_share == (int)order.size() ? lanes : std::max(2, lanes - 1);
    std::vector<std::vector<int>> units;
    std::vector<int> unit_of(rows.size(), -1);
    int rows_open = 0;
    for (int k : order) {
        if (!can_share[k]) continue;
        if (units.empty() || (int)units.back().size() >= together || rows_open + rows[k] > kSharedRows) {
            units.emplace_back();
            rows_open = 0;
        }
        unit_of[k] = (int)units.size() - 1;
        units.back().push_back(k);
        rows_open += rows[k];
    }
    PassUnits p;
    for (int k : order)
        if (unit_of[k] < 0 || units[unit_of[k]].size() < 2) p.alone.push_back({k});
    for (auto& u : units)
        if (u.size() > 1) p.shared.push_back(std::move(u));
    p.beside.resize(p.shared.size());
    int most = 0;
    for (size_t u = p.shared.size(); u-- > 0;) {
        most = std::max(most, (int)p.shared[u].size());
        p.beside[u] = lanes - most;
    }
    return p;
}

size_t gemm_partial_rows_bound(int n_max)
{
    // up to kSweepMaxRows rows: at most kSmallMaxKsplit slices; the block kernel: 4 up to kBlockRows4 rows, 2 up to
    // kBlockRows2
    const size_t n = (size_t)std::max(n_max, 1);
    size_t need = n;
    need = std::max(need, (size_t)kSmallMaxKsplit * std::min<size_t>(n, (size_t)kSweepMaxRows));
    need = std::max(need, (size_t)4 * std::min<size_t>(n, (size_t)kBlockRows4));
    need = std::max(need, (size_t)2 * std::min<size_t>(n, (size_t)kBlockRows2));
    return need;
}

}  // namespace ss
