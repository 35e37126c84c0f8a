// Batched dynamic program for the constrained layer-wise compression problem on gfx950.
//
// Sec. 3.2 (Eq. 2-3) and App. A (Alg. 1) define the computation; include/spdy_dp.h states the
// arithmetic contract (fp32, one add per update, smallest level / smallest t win ties).
//
// Mapping.  Alg. 1's triple loop (layer, level, time) is a min-plus recurrence with no reuse of a
// D_{l-1} element across levels (every level shifts the row by a different tau), so there is no
// contraction to put on the matrix cores: the work per (l, s, t) is one LDS read, one fp32 add
// and a min (plus a compare and a select when the level itself is tracked).  The remark after
// Alg. 1 (vectorise over t by shifting the row) is what the lanes do here:
//   * a prepare kernel subtracts each layer's smallest time from the layer and from the budget
//     (rows shrink to B - M + 1 buckets), bounds the reachable part of each row and fixes the
//     order in which the levels of a layer are visited;
//   * the row of D of a candidate stays in LDS for the whole solve, with a +inf apron of one
//     group width on its left, so a level whose shift falls inside a group of buckets needs no
//     per-lane bounds test; levels whose shift lies beyond the group are never visited;
//   * the time axis is cut into chunks of 64 buckets; a wave keeps a group of R chunks in
//     registers (running minimum, and the level when tracked) and sweeps the layer once; lane i
//     holds the i-th entry of the layer (a level, or with the D record all levels of one shift,
//     which one update serves) and ballots find the applicable entries, whose shifts and errors
//     v_readlane moves to scalar registers or, below, come from LDS two entries at a time;
//   * when D itself is recorded and a layer has at most 64 levels, a lane takes four consecutive
//     buckets and reads them with one aligned ds_read_b128 (twice the LDS bytes per clock of
//     narrower reads on this chip); entries are visited by their shift modulo four, and the minima
//     are kept shifted by that, so that no add needs a word from another lane (sweep_layer);
//   * the level record, and the D record of more than 64 levels, have four buckets a lane that lie a
//     quarter of the row apart, side by side in LDS, where there are two workgroups to a unit (dp_columns).
//     Otherwise, and in short rows of few levels (sweep_tails), lane i works on bucket 64*c + i of a
//     chunk: every ds_read_b32 of the shifted row touches 64 consecutive dwords (conflict-free for
//     any shift);
//   * the waves of a workgroup are split at run time into teams, one candidate per team, so
//     that each wave owns as many chunks as its registers hold whatever the reduced row length
//     is; when every wave holds all its chunks of the row in registers the row is updated in
//     place (one row per candidate), otherwise two rows alternate;
//   * two workgroups of eight waves share a compute unit, and in a launch of one or two rounds
//     of workgroups they take turns at the instruction priority, so that neither runs on the
//     other's leftovers and then alone;
//   * a compute unit wants about sixteen waves of this loop, each with a long group.  Where the
//     usual shape does not give that, a D-record workgroup has sixteen waves: with no more
//     candidates than compute units the second eight divide each layer's ENTRIES with the first
//     eight on the same chunks; a row too long for eight waves' registers is updated in place by
//     sixteen waves with up to the whole LDS of the unit.
// A row that is longer still lives in global memory (two alternating rows per candidate) and is
// computed tile by tile, the part of the previous row a tile reads being staged in LDS first.
#include <hip/hip_runtime.h>

#include <stddef.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "spdy_dp.h"

// Workspace of spdy_dp_solve_batched_static: device memory that belongs to the loaded code
// object, so the entry point never allocates.  In host code this name is only a handle for
// hipGetSymbolAddress; the address the kernels get is looked up once per device.
static __device__ __align__(256) unsigned char scratch[SPDY_DP_STATIC_WORKSPACE_BYTES];

namespace {

constexpr int kWave = 64;            // lanes per wavefront = buckets per chunk
// The fill kernel's shape per record variant.  D record: 8 waves of up to 128 registers, each
// keeping up to 26 chunks of a row (two workgroups, 16 waves, per compute unit): long sweeps
// between the barriers of a layer.  Level record: 16 waves of up to 64 registers with up to 10
// chunks each (value and level per chunk).
constexpr int kMaxGroup = 26;        // most chunks a wave keeps in registers at once (D record)
constexpr int kMaxGroupLevel = 10;   // same when the level is tracked too
// In the instantiation for small batches (kTurns) a wave keeps up to 28: a row of 105 - 112
// chunks (the paper's own sizes, T = 10^4) then still splits into two teams of four waves.  The
// other instantiation stays at 26: with 28 its inner loops are the same instruction for
// instruction, but stress_k256 ran 5 % slower (code placement), and long launches gain nothing.
constexpr int kMaxGroupTurns = 28;
template <bool kLevel, bool kTurns> constexpr int group_limit()
{
    return kLevel ? kMaxGroupLevel : (kTurns ? kMaxGroupTurns : kMaxGroup);
}
// Level record: least levels per layer for comparisons that two levels share.  Finding out which of the two
// it was costs every cell two lane exchanges, a read and an add; below some 14 levels that is more than
// the comparisons saved.  K = 1024, L = 52, B = 10000, us a solve with and without: S = 2 217 and 181,
// S = 8 298 and 274, S = 12 425 and 413, S = 16 471 and 477, S = 40 774 and 901.
constexpr int kPairsFrom = 14;
constexpr int kFillWaves = 8;        // waves of a fill workgroup (D record)
constexpr int kFillWavesLevel = 16;  // (level record)
constexpr int kMaxFillWaves = 16;
template <bool kLevel> constexpr int fill_waves() { return kLevel ? kFillWavesLevel : kFillWaves; }
constexpr int kPriorityTurn = 13;    // log2 of the 100 MHz ticks a workgroup keeps the priority
constexpr int kWalkThreads = 256;    // D-record walk back: 4 waves = 4 candidates per workgroup
constexpr int kLdsStatic = 8192 + 256;    // the fill kernel's static LDS (entry tables, argmin)
constexpr int kLdsBytes = 160 * 1024 - kLdsStatic;       // dynamic LDS a workgroup can get
constexpr int kLdsHalf = 80 * 1024 - kLdsStatic;         // lets two workgroups share a compute unit
// +inf apron left of every row: a group's width, plus one chunk because the 128-bit reads of the
// sweep start one lane (four buckets) below the group
constexpr int kHalo = kMaxGroupTurns * kWave + kWave;
// The longest row the waves of a workgroup can hold in registers (and so update in place), with
// its apron, fits the smaller LDS allocation for either record, and two rows that are any longer
// do not: the in-place case and the launch with the smaller allocation coincide.
constexpr bool kInPlaceFits =
    (kFillWaves * kMaxGroupTurns * kWave + kHalo) * 4 <= kLdsHalf &&
    (kFillWavesLevel * kMaxGroupLevel * kWave + kHalo) * 4 <= kLdsHalf &&
    2 * (kFillWaves * kMaxGroup * kWave + kWave + kHalo) * 4 > kLdsHalf &&
    2 * (kFillWavesLevel * kMaxGroupLevel * kWave + kWave + kHalo) * 4 > kLdsHalf;
static_assert(kInPlaceFits, "path 1 must be exactly the in-place case");
constexpr int kBatch = 8;                 // level tables are padded to a multiple of this
// The 128-bit sweep (see fill_group_quads): a group of R chunks of 64 buckets is quad_chunks(R) quad chunks
// and tail_chunks(R) ordinary ones.
constexpr int kQuadLanes = kWave - 1;             // lanes of a quad chunk that own buckets
constexpr int kQuadChunk = 4 * kQuadLanes;        // 252 buckets
__host__ __device__ constexpr int quad_chunks(int R) { return R * kWave / kQuadChunk; }
__host__ __device__ constexpr int tail_chunks(int R)
{
    return (R * kWave - quad_chunks(R) * kQuadChunk + kWave - 1) / kWave;
}
// What a group of R chunks costs, a quad chunk being 4: a tail chunk has a quarter of the adds and minima, and
// half of the LDS time, its reads being a fourth as wide at half the rate.
__host__ __device__ constexpr int sweep_cost(int R) { return 4 * quad_chunks(R) + 2 * tail_chunks(R); }
// A share of whole quad chunks from bucket t on, as a word of the header (0: the share is what the chunk
// boundaries say).  K = 1024, L = 54, S = 40, B = 10^4: 20 quad chunks instead of 80 chunks, which were 20 quad chunks
// and as many tail chunks as waves: 434 us a solve and 428; parameters as cost: 642 and 600.
constexpr int kMaxQuads = kMaxGroupTurns * kWave / kQuadChunk;
__host__ __device__ constexpr int quad_share(int t, int quads)
{
    return 1 << 30 | quads << 20 | t / 4;
}
static_assert(kMaxFillWaves * kMaxGroupTurns * kWave / 4 < 1 << 20, "rows updated in place");
// Or a share of ordinary chunks alone, where a wave has few of them and few levels (see sweep_tails): up to
// kFewChunks, and kFewUpdates of levels and chunks.  us a solve with quad chunks and entries from LDS, and so:
// K = 1500, L = 66, S = 8, B = 300 149 and 131, B = 586 163 and 138; K = 400, L = 60, B = 1500 147 and 123;
// S = 20, K = 1500, B = 586 172 and 151, K = 1200, L = 93, B = 1132 261 and 231; S = 40, K = 1500, B = 300 180
// and 162.  Of 254 calls around the line none is more than 0.7 % slower; with twice the updates S = 32 and 40
// are up to 4 %.
constexpr int kFewChunks = 6, kFewUpdates = 120;
__host__ __device__ constexpr int tail_share(int t, int chunks)
{
    return quad_share(t, chunks > 0 ? kMaxQuads + chunks : 0);
}
static_assert(kMaxQuads + kFewChunks < 1 << 4, "four bits of the word");
constexpr unsigned kNoLevel = 0xFF;
constexpr size_t kAlign = 256;
constexpr int kMetaHeader = 20;      // int32 words before the per-layer arrays
// meta: header | m_l [L] | chunks of row l [L] | chunk boundaries of the team waves [L][stride]
//       | largest usable shift of layer l [L]
constexpr int kRangeStride = kMaxFillWaves + 1;
// shares of one kind of chunk, behind the boundaries of the usual workgroup's waves
constexpr int kWholeWord = kFillWaves + 1;
static_assert(kWholeWord + kFillWaves <= kRangeStride, "words of a layer");

// kMetaPath: 0 = rows in global memory, 1 / 2 = rows in LDS, fill kernel launched with the
// smaller / larger LDS allocation, 3 = one row in LDS updated in place by a workgroup of twice
// the waves that has a compute unit's LDS to itself (D record; rows too long for path 1),
// 4 = rows in global memory, a workgroup of twice the waves (D record).
// kMetaTeamWaves x kMetaTeams <= waves of a fill workgroup.
// kMetaInPlace: every wave of a team holds all its chunks of a row in registers, so one row per
// candidate suffices (written back between two barriers); otherwise two rows alternate.
enum MetaWord {
    kMetaBudget = 0, kMetaMinTime = 1, kMetaRow = 2, kMetaPath = 3, kMetaTeamWaves = 4,
    kMetaTeams = 5, kMetaInPlace = 6,
    kMetaStage = 7,     // bytes of LDS the global-row launch has for the windows of its tiles
    // what the choice of the path was made from (read back by tests, not by the kernels)
    kMetaWaves = 8,     // waves of a fill workgroup
    kMetaMaxGroup = 9,  // most chunks a wave keeps in registers
    kMetaLdsSmall = 10, // dynamic LDS bytes of the in-place launch
    kMetaLdsLarge = 11, // dynamic LDS bytes of the two-row launch (0: not enqueued)
    kMetaHalo = 12,     // floats of the +inf apron left of a row
    kMetaSplit = 13,    // 1: the in-place launch has twice kMetaWaves waves (see dp_fill, kSplit)
    kMetaWideWaves = 14, // waves of the wide in-place launch (0: not enqueued)
    kMetaWideGroup = 15, // most chunks one of its waves keeps in registers
    kMetaLdsWide = 16,   // its dynamic LDS bytes
    kMetaGlobalWaves = 17, // waves of the global-row launch
    kMetaTable = 18,    // 1: the call leaves the whole table in the record (0: scratch)
    // > 0: dp_tiles or dp_wide does the work (see there), not the launch of kMetaPath; < 0: dp_columns, and not
    // dp_fill, is the launch of path 1 (see there), the buckets of a position negated
    kMetaTiles = 19
};

enum Variant { kValueRecord = 0, kLevelRecord = 1 };

// dp_columns (see there): chunks of 64 positions that a wave holds at most, and of 64 buckets where the row is not
// folded; candidates of a workgroup at most; entries that are read behind the last of a table, and not used.
enum Columns { kNoColumns = 0, kValueColumns = 1, kLevelColumns = 2 };       // which record it is enqueued for
template <bool kLevel> constexpr int column_chunks() { return kLevel ? 5 : 7; }
constexpr int kPlainChunks = 6;
constexpr int kFoldLevels = 16, kFoldBudget = 800, kFoldWork = 300;   // least, level record
constexpr int kColumnTeams = 8;
constexpr int kLookAhead = 4;
// Waves of a team, a power of two, and the chunks of `n` that the one with the most has.
__device__ __forceinline__ int column_waves(int teams) { return teams == 1 ? 8 : (teams == 2 ? 4 : (teams <= 4 ? 2 : 1)); }
static_assert(kFillWaves == 8, "column_waves");
__device__ __forceinline__ int column_share(int n, int tw) { return (n + tw - 1) >> __builtin_ctz(tw); }
// Whether a row of `n` chunks is better not folded, `tw` waves to a row: where whole chunks of positions are more
// than what the wider reads save.
__device__ __forceinline__ bool plain_is_better(int n, int tw)
{
    const int plain = column_share(n, tw), folded = column_share((n + 3) / 4, tw);
    return plain <= kPlainChunks && 40 * folded > 14 * plain;
}
// Floats of LDS: of a candidate's row, ghost or apron included, and with its entries of two layers.
__device__ __forceinline__ int column_row(int n, int tw, bool plain)
{
    const int n4 = (n + 3) / 4;
    return plain ? (n + column_share(n, tw)) * kWave : 4 * (kWave * (n4 + column_share(n4, tw)) + 1);
}
__device__ __forceinline__ int column_entries(int S) { return (S + kWave - 1) / kWave * kWave + kLookAhead; }
__device__ __forceinline__ int column_floats(int n, int tw, bool plain, int S, bool level)
{
    return column_row(n, tw, plain) + 2 * (level ? 3 : 2) * column_entries(S);
}
// What the fill of rows of `n` chunks costs with `teams` of them to a workgroup, in chunks of positions that are
// swept; infinite where they do not have the LDS or the registers.  `slots`: workgroups the chip holds at once.
// Rounds of workgroups times what a workgroup has to do, where a rest that finds every workgroup a compute unit to
// itself is 0.7 of a round, a chunk of buckets 0.35 of one of positions, a wave's own share counts besides (its reads
// wait for each other) and so does what every layer takes.  Only compared with itself.  D record: the same for
// every number that there is room for.
__device__ __forceinline__ float column_cost(int K, int n, int S, bool level, int slots, int teams)
{
    const int most = level ? column_chunks<true>() : column_chunks<false>();
    const int tw = column_waves(teams), n4 = (n + 3) / 4;
    const bool plain = plain_is_better(n, tw);
    if (teams > 1 && ((!plain && column_share(n4, tw) > most) ||
                      teams * column_floats(n, tw, plain, S, level) * (int)sizeof(float) > kLdsHalf))
        return __builtin_inff();
    if (!level)
        return 0.0f;
    const float row = plain ? 0.35f * n : n4, share = plain ? 0.35f * column_share(n, tw) : column_share(n4, tw);
    // (whole numbers by fp32 divisions: integer ones took 1 us)
    const float groups = floorf((K + (teams - 0.5f)) / teams), full = floorf((groups + 0.5f) / slots);
    const float rest = groups - full * slots;
    const float rounds = full + (rest < 0.5f ? 0.0f : (2.0f * rest > slots ? 1.0f : 0.7f));
    return rounds * (8.0f + teams * row + 4.0f * share);
}
// Teams of a workgroup, at most `teams`: as many as there is room for, or fewer where these cost less by a twentieth.
// (As many as there is room for are often a few more than one round of workgroups takes, and the second round takes
// nearly as long.)  us a fill with the most and so, L = 16: S = 128, K = 3000, 17 chunks 885 (5 teams) and 610 (4),
// K = 4000, 19 chunks 1190 and 811; S = 40, K = 4000, 13 chunks 285 (6) and 235 (4), K = 2100, 25 chunks 253 (4) and
// 245 (3).  Of 624 fills none was more than 0.1 % slower.
// `cost`: column_cost of 1, 2, ... teams.
__device__ __forceinline__ int plan_columns(const float *cost, int teams)
{
    float of[kColumnTeams], limit = __builtin_inff();
#pragma unroll
    for (int i = 0; i < kColumnTeams; ++i)       // (read together)
        of[i] = cost[i];
    int best = 0;
#pragma unroll
    for (int i = kColumnTeams; i > 0; --i)
        if (i <= teams && of[i - 1] < limit) {
            limit = best == 0 ? 0.95f * of[i - 1] : of[i - 1];
            best = i;
        }
    return best;
}
// one team: any row that a workgroup of either record may have in place, with all the entries there may be
static_assert(kFillWavesLevel * kMaxGroupLevel <= 4 * kFillWaves * column_chunks<true>() &&
                  kFillWaves * kMaxGroupTurns <= 4 * kFillWaves * column_chunks<false>() &&
                  (4 * (kWave * (kFillWaves + 1) * column_chunks<false>() + 1) + 2 * 3 * (256 + kLookAhead)) * 4 <=
                      kLdsHalf, "rows in place fit dp_columns");


// ---------------------------------------------------------------------------------------------
// Workspace layout (host side, shared by every entry point)
struct Layout {
    int status;
    int variant;
    size_t row;          // buckets per padded row for the full budget (multiple of 64)
    bool may_spill;      // rows of the full budget may exceed LDS: the global-row launch is needed
    size_t s8;           // levels per layer padded to a multiple of kBatch
    size_t meta_off;     // int32 meta[kMetaHeader + (3 + kRangeStride) L]
    size_t shifts_off;   // int32 shifts[L][s8]: tau - m_l of the r-th visited entry
    size_t order_off;    // int32 order[L][s8]: level index at position r of the visiting order
    size_t start_off;    // int32 start[L][s8 + kBatch]: first position of entry r (D record)
    size_t entry_off;    // int32 entry[L][s8]: the entry that level s belongs to (D record)
    size_t tstar_off;    // int32 tstar[K]
    size_t record_off;   // float D[K][L][row]  or  uint8 P[K][L][row]
    size_t rows_value;   // float rows[K][2][kHalo + row] after the record, when may_spill
    size_t rows_level;
    size_t total_value;  // bytes needed by the D-record variant
    size_t total_level;  // bytes needed by the level-record variant
};

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

// `workspace_bytes` selects the variant; pass SIZE_MAX to get the sizes only.  `rec_rows`: rows
// of the record per candidate (L, or fewer for the solve with checkpoints).
Layout make_layout(int K, int L, int S, int B, size_t workspace_bytes, long long rec_rows = -1)
{
    Layout lay{};
    if (K <= 0 || L <= 0 || S <= 0 || B < 0) {
        lay.status = SPDY_DP_ERR_DIM;
        return lay;
    }
    if (S > 255) {
        lay.status = SPDY_DP_ERR_LEVELS;
        return lay;
    }
    if (B > INT32_MAX - 2 * kWave * kMaxGroupTurns) {   // bucket indices are int32 on the device
        lay.status = SPDY_DP_ERR_OVERFLOW;
        return lay;
    }
    lay.row = align_up((size_t)B + 1, kWave);
    const unsigned __int128 cells = (unsigned __int128)K * ((unsigned __int128)L + 2) *
                                    (lay.row + kHalo);
    if (cells * sizeof(float) + (unsigned __int128)K * 16 + (unsigned __int128)L * 4096 >
        (unsigned __int128)1 << 62) {
        lay.status = SPDY_DP_ERR_OVERFLOW;
        return lay;
    }
    const size_t row_bytes = (lay.row + kHalo) * sizeof(float);
    lay.may_spill = 2 * row_bytes > (size_t)kLdsBytes;
    lay.s8 = align_up((size_t)S, kBatch);
    lay.meta_off = 0;
    lay.shifts_off =
        align_up((kMetaHeader + (3 + (size_t)kRangeStride) * L) * sizeof(int32_t), kAlign);
    lay.order_off = align_up(lay.shifts_off + (size_t)L * lay.s8 * sizeof(int32_t), kAlign);
    lay.start_off = align_up(lay.order_off + (size_t)L * lay.s8 * sizeof(int32_t), kAlign);
    lay.entry_off =
        align_up(lay.start_off + (size_t)L * (lay.s8 + kBatch) * sizeof(int32_t), kAlign);
    lay.tstar_off = align_up(lay.entry_off + (size_t)L * lay.s8 * sizeof(int32_t), kAlign);
    lay.record_off = align_up(lay.tstar_off + (size_t)K * sizeof(int32_t), kAlign);
    const size_t rows = lay.may_spill ? 2 * (size_t)K * row_bytes : 0;
    const size_t nrec = rec_rows < 0 ? (size_t)L : (size_t)rec_rows;
    lay.rows_value = align_up(lay.record_off + (size_t)K * nrec * lay.row * sizeof(float), kAlign);
    lay.rows_level = align_up(lay.record_off + (size_t)K * nrec * lay.row, kAlign);
    lay.total_value = lay.rows_value + rows;
    lay.total_level = lay.rows_level + rows;
    if (workspace_bytes >= lay.total_value)
        lay.variant = kValueRecord;
    else if (workspace_bytes >= lay.total_level)
        lay.variant = kLevelRecord;
    else {
        lay.status = SPDY_DP_ERR_WORKSPACE;
        return lay;
    }
    lay.status = SPDY_DP_OK;
    return lay;
}

#include "wave_ops.h"

// ---------------------------------------------------------------------------------------------
// Sum of `v` over a workgroup of 256 threads (returned to every thread); if `exclusive` is given
// it receives the sum over the threads before this one.  part: 8 words of LDS.
__device__ __forceinline__ long long block_scan_256(long long v, long long *part,
                                                    long long *exclusive)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const long long incl = wave_scan(v, 0ll, Add{});
    __syncthreads();                              // part may still be read from a previous call
    if (lane == kWave - 1)
        part[wave] = incl;
    __syncthreads();
    long long before = 0, total = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const long long p = part[w];
        before += w < wave ? p : 0;
        total += p;
    }
    if (exclusive)
        *exclusive = before + incl - v;
    return total;
}

// What the prepare kernel plans the tiles of a row with (see dp_tiles.h).
struct TileArgs {
    int units;               // compute units
    int only_memory;         // 1: only where rows would lie in memory
    int most;                // tiles of a row at most (0: dp_tiles is not enqueued)
    int lds;                 // floats of its LDS
    int *books;              // ticket, keys and counters of the tiles
    int room;                // their words
};

constexpr int kTileWaves = 16;
constexpr int kTileChunks = 7;       // short tiles: chunks a wave takes at most
constexpr int kTileUnits = 6;        // long tiles: quad chunks a wave takes at most
constexpr int kTileMost = 16;        // tiles of a row at most
constexpr int kTileLayers = 8;       // layers whose entries have to fit LDS at once
constexpr int kTileBuckets = 252;    // buckets of a quad chunk
// what kMetaTiles holds: tiles | kTileLong | quads of the apron << 12
constexpr int kTileLong = 1 << 11;
// books: ticket | - | key of every tile [K][tiles] (two words) | counters of every tile [K][tiles][4]:
//        rows in memory (short tiles: up to the last even one, up to the last odd one), -, done
constexpr int kTileFlags = 4, kTileDone = 3;
__device__ __forceinline__ int *tile_flags(int *books, int solves) { return books + 2 + 2 * solves; }

// Into how many tiles the rows of `chunks` chunks are cut, and of which kind: what is estimated to be
// fastest, one pair per lane; 0 where nothing fits.  One wave.
__device__ __forceinline__ void plan_tiles(int K, int L, int S, int bp, int chunks, int row_chunks,
                                           int span, int mean_span, const TileArgs &ta, int *plan)
{
    const int lane = threadIdx.x & (kWave - 1);
    if (bp < 0 || ta.most == 0) {
        if (lane == 0)
            *plan = bp < 0 && ta.most > 0 && ta.only_memory == 0 ? 1 : 0;
        return;
    }
    const int tiles = (lane & (kTileMost - 1)) + 1;
    const bool is_long = lane >= kTileMost;
    const int grain = is_long ? kTileBuckets : kWave;
    const int apron = (span + 3) / 4 + 2;         // quads
    const int all = (chunks * kWave + grain - 1) / grain;
    const int units = (all + tiles - 1) / tiles;
    const int waves = is_long ? kTileWaves : kTileWaves - (tiles > 1 ? 4 : 2);
    const int mine = (units + waves - 1) / waves;
    const int s8 = (S + kBatch - 1) / kBatch * kBatch;
    const long long lines = (is_long ? 1 : 2) * (4LL * apron + (long long)units * grain);
    const bool fits = tiles <= ta.most && (tiles - 1) * units < all && lane < 2 * kTileMost &&
                      mine <= (is_long ? kTileUnits : kTileChunks) && (!is_long || S <= kWave) &&
                      (tiles == 1 || (long long)K * tiles * (2 + kTileFlags) + 2 <= ta.room) &&
                      apron < 1 << 20 &&
                      lines + min(L, kTileLayers) * (2LL * s8 + 1) + 4 <= ta.lds;
    // Clocks, fitted to measured fills (a lone S = 40 candidate of 4955 buckets in 1, 2, 4, 8 short
    // tiles: 8400, 5900, 3700, 2900 a layer; one of 49581 in 3, 4, 6, 8 long ones, with a sweep that took a
    // seventh longer than the present one: 26300, 21000, 17300, 13000).
    // A SIMD issues an instruction every four clocks or so, whichever of its waves it is from.
    const float pairs = 0.42f * S;                // entries are fewer than levels
    const float of_simd = (float)((units + 3) / 4), waves_of_simd = (float)((min(waves, units) + 3) / 4);
    // (A wave brings a short tile's apron, and all tiles on all compute units slow the memory down; of long
    // tiles 21200 and 25700 clocks a layer.)
    const bool crowded = 2 * K * tiles > ta.units;
    const float bring = tiles == 1 ? 0.0f : mean_span * (crowded ? 2.0f : 1.2f);
    const float layer =
        is_long ? (1500.0f + fmaxf(4.2f * pairs * (of_simd * 17.5f + waves_of_simd * 12.0f),
                                   13.0f * pairs * (mine * 17.5f + 12.0f))) *
                      (crowded ? 1.25f : 1.0f)    // (the second: a wave by itself)
                : 700.0f + bring +
                      4.2f * (of_simd * pairs * 4.9f + waves_of_simd * (pairs * 3.0f + 50.0f));
    // what a tile is behind the one below it: more with more workgroups at the same memory
    const float lag = 1.5f * layer + 3000.0f + 60.0f * min(K * tiles, ta.units);
    const float rounds = (float)((K * tiles + ta.units - 1) / ta.units);
    float clocks = rounds * L * layer + (tiles - 1) * lag;
    clocks = fits ? clocks : __builtin_inff();
    float best = clocks;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1)
        best = fminf(best, __shfl_xor(best, off, kWave));
    const unsigned long long set = __ballot(fits && clocks == best);
    // Rows in memory, one workgroup per candidate: 21 updates a clock.  ms a solve of L = 54, S = 40 so and in
    // tiles, B = 10^5: K = 140 1.50 and 1.18, K = 200 1.56 and 1.77, K = 300 3.14 and 2.34, K = 512 3.47 and
    // 3.68, K = 1000 6.87 and 7.01; B = 60000: 1.04 and 0.83, 1.07 and 0.97 (not taken), 2.05 and 1.60, 2.16
    // and 2.21, 4.31 and 4.21.
    const float untiled = (float)((K + ta.units - 1) / ta.units) * L *
                          (1500.0f + row_chunks * pairs * 6.15f);
    const bool tiled = set != 0 && (ta.only_memory == 0 || best < untiled);
    if (lane == 0 && !tiled)
        *plan = 0;
    if (tiled && lane == __builtin_ctzll(set))
        *plan = tiles | (is_long ? kTileLong : 0) | apron << 12;
}

// Prepare, workgroup 0: per-layer smallest time m_l, M = sum m_l, reduced budget B - M, and how
// many 64-bucket chunks of each reduced row can hold a finite value (the largest reachable
// reduced time after layer l is sum_{j<=l} max_s (tau[j][s] - m_j) over the levels that fit the
// reduced budget).  It also picks the path: which launch of the fill kernel (LDS allocation
// lds_small or lds_large bytes, `waves` waves per workgroup) fits, into how many teams its waves
// split, and whether one row per candidate is enough; and it records each layer's largest usable
// shift (the tiles of the global-row path size their window in LDS by it).  Thread i owns layers i,
// i + 256, ...; a layer's times are read by eight lanes.
// What bounds it: latency, about 11000 clocks of dependent steps for L = 54, S = 40.
__device__ void prepare_budget(const int32_t *__restrict__ tau, int K, int slots, int L, int S,
                               int B, int waves, int max_group, int lds_small, int lds_large,
                               int lds_stage, int split, int wide_waves, int wide_group,
                               int lds_wide, int global_waves, bool quads, bool tails, int columns, const TileArgs &ta,
                               int32_t *words, int32_t *__restrict__ meta)
{
    __shared__ long long s_sum[8];
    __shared__ int s_span[4], s_team_waves, s_tiles, s_beyond, s_whole;
    __shared__ float s_columns[kColumnTeams];
    int32_t *const s_least = words, *const s_most = words + 256;
    const int tid = threadIdx.x;
    if (tid == 0)
        s_beyond = 0;
    int32_t *mn = meta + kMetaHeader;
    int32_t *nact = meta + kMetaHeader + L;
    int32_t *spans = meta + kMetaHeader + (2 + (size_t)kRangeStride) * L;
    const int lane = tid & (kWave - 1), wave = tid / kWave;

    // Least and largest time of the layers [base, base + n), or (kCapped) the largest that is not above
    // the layer's word of s_least (nothing where that is negative).  Eight lanes per layer, so that all
    // loads of 32 layers are on their way at once and three steps across lanes join them: L = 54 takes
    // 2000 clocks (a wave per layer, four or eight layers at a time: 4800 and 7400, most of it scans).
    // The second reading costs 1000; by one thread, a level after the other, it made the shortest
    // fills 1.15 of what they are (K = 1, L = 8, S = 40, B = 500: 27.5 us and 24.6).
    auto read_times = [&](int base, int n, auto capped) __attribute__((always_inline)) {
        constexpr bool kCapped = decltype(capped)::value != 0;
        constexpr int kLanes = 8, kLoads = 8;
        const int part = lane & (kLanes - 1);
        for (int i0 = wave * (kWave / kLanes); i0 < n; i0 += 256 / kLanes) {
            const int i = i0 + lane / kLanes, at = min(i, n - 1);
            const int32_t *const tau_i = tau + (size_t)(base + at) * S;
            const int cap = kCapped ? s_least[at] : INT32_MAX;
            if (kCapped && !__any(cap >= 0))
                continue;
            int least = INT32_MAX, most = 0;
            for (int s0 = 0; s0 < S; s0 += kLanes * kLoads) {
                int v[kLoads];
#pragma unroll
                for (int q = 0; q < kLoads; ++q)  // (past the last level: that one once more)
                    v[q] = tau_i[min(s0 + q * kLanes + part, S - 1)];
#pragma unroll
                for (int q = 0; q < kLoads; ++q) {
                    least = min(least, v[q]);
                    most = v[q] <= cap ? max(most, v[q]) : most;
                }
            }
            if (!kCapped)
                least = group_join(least, kLanes, Smaller{});
            most = group_join(most, kLanes, Larger{});
            if (part == 0 && i < n) {
                if (!kCapped)
                    s_least[i] = least;
                s_most[i] = most;
            }
        }
        __syncthreads();
    };

    long long local = 0;
    int m_first = 0, most_first = 0;              // of the first block of layers: not read again
    for (int base = 0; base < L; base += 256) {
        const int n = min(256, L - base);
        read_times(base, n, Many<0>{});
        if (tid < n) {
            const int m = s_least[tid], most = s_most[tid];
            mn[base + tid] = m;
            spans[base + tid] = most;             // (the largest time, for now)
            local += m;
            if (base == 0) {
                m_first = m;
                most_first = most;
            }
        }
        __syncthreads();
    }
    const long long M = block_scan_256(local, s_sum, nullptr);
    const int bp = (M > B) ? -1 : (int)(B - M);
    int widest = 0;
    long long reach = 0;                          // sum of the spans of the layers so far
    for (int base = 0; base < L; base += 256) {
        const int l = base + tid;
        int m = 0, span = 0, cap = -1;
        if (l < L && bp >= 0) {
            m = base == 0 ? m_first : mn[l];
            span = (base == 0 ? most_first : spans[l]) - m;
            cap = span > bp ? m + bp : -1;        // (at most B)
        }
        s_least[tid] = cap;
        if (cap >= 0)
            s_beyond = 1;
        __syncthreads();
        if (s_beyond != 0) {                      // some level is beyond the budget: once more without
            read_times(base, min(256, L - base), Many<1>{});
            span = cap >= 0 ? s_most[tid] - m : span;
        }
        long long h = 0;                          // sum over the layers of this block before this one
        const long long total = block_scan_256(span, s_sum, &h);
        if (l < L) {
            h += reach + span;
            const long long top = h < bp ? h : bp;
            nact[l] = bp < 0 ? 0 : (int)((top + kWave) / kWave);
            spans[l] = span;
        }
        reach += total;
        widest = max(widest, span);
    }
    // (256 threads' atomics on one word of LDS took 5000 clocks here: every call 1.7 us longer)
    widest = wave_scan(widest, 0, Larger{});
    if (lane == kWave - 1)
        s_span[wave] = widest;
    __syncthreads();
    const long long top = reach < bp ? reach : bp;
    const int last_chunks = bp < 0 ? 0 : (int)((top + kWave) / kWave);     // of the last row
    if (tid < kWave)
        plan_tiles(K, L, S, bp, last_chunks, (bp + kWave) / kWave,
                   max(max(s_span[0], s_span[1]), max(s_span[2], s_span[3])), (int)(reach / L), ta,
                   &s_tiles);
    else if (columns != kNoColumns && tid < kWave + kColumnTeams)
        s_columns[tid - kWave] =
            column_cost(K, min(last_chunks, 1 << 12), S, columns == kLevelColumns, slots, tid - kWave + 1);
    __syncthreads();
    if (tid == 0) {
        const int rowp = bp < 0 ? 0 : (bp + kWave) / kWave * kWave;
        meta[kMetaBudget] = bp;
        meta[kMetaMinTime] = M > INT32_MAX ? INT32_MAX : (int)M;
        meta[kMetaRow] = rowp;
        int path = 1, teams = 1, inplace = 0;     // an infeasible table is reported by path 1
        int plan_waves = waves;                   // waves of the launch that does the work
        if (bp >= 0) {
            const long long one_row = ((long long)rowp + kHalo) * (long long)sizeof(float);
            const int want = (rowp / kWave + max_group - 1) / max_group;   // waves per candidate
            inplace = want <= waves ? 1 : 0;
            // a row updated in place always fits lds_small (kInPlaceFits), so path 1 is exactly
            // the in-place case of a workgroup of `waves` waves
            const long long team_lds = inplace ? one_row : 2 * one_row;
            const int lds = lds_small;
            path = inplace ? 1 : (team_lds <= lds_large ? 2 : 0);
            // a longer row that the waves of the wide launch can still hold in registers, and
            // that fits its LDS, is updated in place there
            if (!inplace && wide_waves > 0 &&
                (rowp / kWave + wide_group - 1) / wide_group <= wide_waves && one_row <= lds_wide) {
                path = 3;
                inplace = 1;
                plan_waves = wide_waves;
            } else if (path == 0 && global_waves > waves) {
                path = 4;                         // the global-row launch of twice the waves
                plan_waves = global_waves;
            } else if (inplace) {
                // as many candidates per workgroup as keeps every wave at <= max_group chunks
                teams = waves / want;
                const long long fit = lds / team_lds;
                if (teams > fit)
                    teams = (int)fit;
                // with fewer candidates than the chip has room for, fewer candidates share a
                // workgroup, so that each gets more waves and finishes sooner
                const int spread = (K + slots - 1) / slots;
                if (teams > spread)
                    teams = spread;
            }
        }
        int cells = 0;                            // of a position
        if (columns != kNoColumns && path == 1) {
            if (bp >= 0)
                teams = plan_columns(s_columns, teams);
            cells = plain_is_better(last_chunks, column_waves(teams)) ? 1 : 4;
            plan_waves = waves = kFillWaves;
            max_group = 4 * (columns == kLevelColumns ? column_chunks<true>() : column_chunks<false>());
        }
        meta[kMetaPath] = path;
        meta[kMetaTeams] = teams;
        meta[kMetaTeamWaves] = plan_waves / teams;
        meta[kMetaInPlace] = inplace;
        meta[kMetaStage] = lds_stage;
        meta[kMetaWaves] = waves;
        meta[kMetaMaxGroup] = max_group;
        meta[kMetaLdsSmall] = lds_small;
        meta[kMetaLdsLarge] = lds_large;
        meta[kMetaHalo] = kHalo;
        meta[kMetaSplit] = split;
        meta[kMetaWideWaves] = wide_waves;
        meta[kMetaWideGroup] = wide_group;
        meta[kMetaLdsWide] = lds_wide;
        meta[kMetaGlobalWaves] = global_waves;
        s_team_waves = plan_waves / teams;
        // (not with a second half of waves, which leave their share of a bucket's minimum in one place)
        s_whole = path == 1 && quads && split == 0 ? 1 : 0;
        if (ta.only_memory != 0 && path != 0 && path != 4)
            s_tiles = 0;
        meta[kMetaTiles] = cells ? -cells : s_tiles;
    }
    __syncthreads();
    const int tw = s_team_waves;
    if (const int tiles = s_tiles & 0xFF; tiles > 1) {
        int *const flags = tile_flags(ta.books, K * tiles);
        for (int i = tid; i < K * tiles * kTileFlags; i += 256)
            flags[i] = 0;
        if (tid == 0)
            ta.books[0] = 0;
    }
    const bool whole_quads = s_whole != 0;
    for (int l = tid; l < L; l += 256) {
        // wave w of a team sweeps chunks [w n / tw, (w + 1) n / tw) of this row
        const int n = nact[l];
        int32_t *range = meta + kMetaHeader + 2 * L + (size_t)l * kRangeStride;
        for (int w = 0; w <= tw; ++w)
            range[w] = (int)((unsigned)(w * n) / (unsigned)tw);   // (16 rows of 2^25 chunks fit)
        // or whole quad chunks, where the wave with the most has less to do that way; the last of
        // them are moved down to the row's end and lie over the ones before
        if (whole_quads) {
            const int units = (n * kWave + kQuadChunk - 1) / kQuadChunk, most = (units + tw - 1) / tw;
            const int chunks = (n + tw - 1) / tw;
            const bool few = tails && chunks <= kFewChunks && S * chunks <= kFewUpdates;
            const bool whole = most <= kMaxQuads && n * kWave >= most * kQuadChunk &&
                               4 * most < sweep_cost(chunks);
            for (int w = 0; w < tw; ++w) {
                const int unit = w * units / tw, mine = (w + 1) * units / tw - unit;
                const int first = min(unit * kQuadChunk, n * kWave - mine * kQuadChunk);
                const int c = range[w], c_end = range[w + 1];
                range[kWholeWord + w] = few ? tail_share(c * kWave, c_end - c)
                                            : (whole ? quad_share(first, mine) : 0);
            }
        }
    }
}

// Prepare, workgroup 1 + l: what the fill visits in layer l, in which order, with the shifts
// tau - m_l; padding up to s8 gets shift INT32_MAX, which no group of buckets can use.
//   level tracked (sorted = 0): one entry per level, ascending in s, so that ties go to the
//     smallest s through the strict "<"; entry r is level r.
//   D record (sorted = 1): the levels are ordered by ascending shift, ties by index, and levels
//     with the SAME shift form one entry: they read the same cell of D_{l-1}, and a rounded add
//     is monotone in the addend, so min_s fl(p + e_s) = fl(p + min_s e_s) bit for bit (up to
//     the sign of a zero): one update with the smallest error of the entry's levels serves them
//     all.  Entry r covers positions start[r] .. start[r + 1] - 1 of `order`, level s belongs
//     to entry entry[s]; the entries a group of buckets can use form a prefix.
//   D record, at most 64 levels (sorted = 2): as above, but the entries are ordered by
//     (shift mod 4, shift): the sweep reads four consecutive buckets per lane with one aligned
//     128-bit LDS read and treats the four residues of the shift separately; the usable entries
//     of a residue then form a prefix of that residue's run.  Nothing reads order and start then;
//     dp_tiles has its books there.
//   D record, where dp_tiles is known to do the work whatever the number of levels (sorted = 3): by
//     shift, and order and start are left alone for the same reason.
// One thread per level (S <= 255).
__device__ void prepare_order(const int32_t *__restrict__ tau, int l, int S, int s8, int sorted,
                              int32_t *__restrict__ shifts, int32_t *__restrict__ order,
                              int32_t *__restrict__ start, int32_t *__restrict__ entry_of,
                              int32_t *words)
{
    int32_t *const s_shift = words, *const s_level = words + 256;
    int32_t *const s_tau = words + 512;           // the layer's times: every thread reads them all
    __shared__ int s_entries;
    const int s = threadIdx.x;
    int32_t *shifts_l = shifts + (size_t)l * s8;
    int32_t *order_l = order + (size_t)l * s8;
    bool twin = false;                            // a later level of the layer takes the same time
    const int mine = s < S ? tau[(size_t)l * S + s] : INT32_MAX;
    s_tau[s] = mine;
    __syncthreads();
    if (s < S) {
        int rank = 0, m = INT32_MAX;
#pragma unroll 8
        for (int o = 0; o < S; ++o)
            m = min(m, s_tau[o]);
        const int residues = sorted == 2 ? 3 : 0;
        const int mine_class = (mine - m) & residues;
#pragma unroll 8
        for (int o = 0; o < S; ++o) {
            const int other = s_tau[o];
            const int other_class = (other - m) & residues;
            const bool before = other_class != mine_class ? other_class < mine_class
                                                          : (other < mine || (other == mine && o < s));
            rank += before ? 1 : 0;
            twin |= o > s && other == mine;
        }
        if (!sorted)
            rank = s;
        if (sorted < 2)
            order_l[rank] = s;
        if (sorted) {
            s_shift[rank] = mine - m;
            s_level[rank] = s;
        } else {
            shifts_l[rank] = mine - m;
        }
    } else if (s < s8 && sorted < 2) {
        order_l[s] = 0;
        if (!sorted)
            shifts_l[s] = INT32_MAX;
    }
    int32_t *start_l = start + (size_t)l * (s8 + kBatch);
    if (!sorted) {
        // level order: start[0..1] holds, for the first 64 levels, the set of those that have
        // such a twin (the only ones that can make a later level not worth visiting)
        const unsigned long long twins = __ballot(twin);
        if (s == 0) {
            start_l[0] = (int32_t)(twins & 0xFFFFFFFFull);
            start_l[1] = (int32_t)(twins >> 32);
        }
        return;
    }
    __syncthreads();
    const int r = threadIdx.x;                    // a position of the sorted order
    if (r < S) {
        int entry = 0;                            // distinct shifts before position r
        for (int o = 1; o <= r; ++o)
            entry += s_shift[o] != s_shift[o - 1] ? 1 : 0;
        if (r == 0 || s_shift[r] != s_shift[r - 1]) {
            shifts_l[entry] = s_shift[r];
            if (sorted < 2)
                start_l[entry] = r;
        }
        entry_of[(size_t)l * s8 + s_level[r]] = entry;
        if (r == S - 1)
            s_entries = entry + 1;
    }
    __syncthreads();
    for (int e = s_entries + r; e < s8 + kBatch; e += 256) {
        if (sorted < 2)
            start_l[e] = S;                       // the last entry ends here; padding is empty
        if (e < s8)
            shifts_l[e] = INT32_MAX;
    }
}

struct PrepareArgs {
    int slots, s8, B, waves, max_group, lds_small, lds_large, lds_stage, sorted, split;
    int wide_waves, wide_group, lds_wide, global_waves, table, tails, columns;
    int32_t *meta, *shifts, *order, *start, *entry_of;
    TileArgs tiles;
};

__device__ __forceinline__ void prepare(const int32_t *__restrict__ tau, int K, int L, int S,
                                        const PrepareArgs &a, int block)
{
    __shared__ int32_t words[3 * 256];
    if (block == 0 && threadIdx.x == 0)
        a.meta[kMetaTable] = a.table;
    if (block == 0)
        prepare_budget(tau, K, a.slots, L, S, a.B, a.waves, a.max_group, a.lds_small, a.lds_large,
                       a.lds_stage, a.split, a.wide_waves, a.wide_group, a.lds_wide,
                       a.global_waves, a.sorted == 2, a.tails != 0, a.columns, a.tiles, words, a.meta);
    else
        prepare_order(tau, block - 1, S, a.s8, a.sorted, a.shifts, a.order, a.start, a.entry_of,
                      words);
}

__global__ __launch_bounds__(256) void dp_prepare(const int32_t *__restrict__ tau, int K, int L,
                                                  int S, PrepareArgs a)
{
    prepare(tau, K, L, S, a, blockIdx.x);
}

// ---------------------------------------------------------------------------------------------
// v_min_f32 / v_min3_f32 without the canonicalising v_max the compiler puts in front of fminf
// (no NaN can occur: err is finite or +inf and D starts at -0 / +inf).
__device__ __forceinline__ void vmin(float &b, float x)
{
    asm("v_min_f32 %0, %0, %1" : "+v"(b) : "v"(x));
}
__device__ __forceinline__ void vmin3(float &b, float x, float y)
{
    asm("v_min3_f32 %0, %0, %1, %2" : "+v"(b) : "v"(x), "v"(y));
}
__device__ __forceinline__ float min3(float x, float y, float z)
{
    float least;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(least) : "v"(x), "v"(y), "v"(z));
    return least;
}

// Where err[k][l][s] comes from: an explicit table, or the product of a per-layer sensitivity
// c[k][l] and a per-level weight w[s] (Eq. 4), formed with one fp32 multiply when it is needed.
struct ErrRow {          // the S errors of one (candidate, layer)
    const float *err_kl; // explicit row, or nullptr
    const float *w;
    float c_kl;
    __device__ __forceinline__ float at(int s) const
    {
        return err_kl ? err_kl[s] : __fmul_rn(c_kl, w[s]);
    }
};
struct ErrSource {
    const float *err;    // [K][L][S], or nullptr
    const float *c;      // [K][L]
    const float *w;      // [S]
    __device__ __forceinline__ ErrRow row(size_t k, int l, int L, int S) const
    {
        ErrRow r;
        r.err_kl = err ? err + (k * L + l) * S : nullptr;
        r.w = w;
        r.c_kl = err ? 0.0f : c[k * L + l];
        return r;
    }
    // The same source seen from candidate k (its [L][S] table or its [L] sensitivities), so that
    // a loop over the layers of one candidate does not redo the 64-bit index arithmetic.
    __device__ __forceinline__ ErrSource of_candidate(size_t k, int L, int S) const
    {
        return ErrSource{err ? err + k * L * S : nullptr, c ? c + k * L : nullptr, w};
    }
    __device__ __forceinline__ ErrRow layer(int l, int S) const   // of a per-candidate view
    {
        ErrRow r;
        r.err_kl = err ? err + (size_t)l * S : nullptr;
        r.w = w;
        r.c_kl = err ? 0.0f : c[l];
        return r;
    }
};

// Re-solving candidates that share their first layers with an already solved incumbent
// (Alg. 4 resamples a few sensitivities of the incumbent): candidate k's tables equal the
// incumbent's for layers < first_layer[k], so its rows of D do too, and the fill starts at
// layer first_layer[k] from the incumbent's recorded row first_layer[k] - 1.
struct Resume {
    const int32_t *first_layer;   // [K] in [0, L], or nullptr: every candidate starts at layer 0
    const float *inc_rec;         // the incumbent's D record, float [L][pitch]
    const int32_t *inc_meta;      // its header: without a whole table there is nothing to resume from
    __device__ __forceinline__ int start(int k, int L) const
    {
        if (!first_layer || !inc_meta[kMetaTable])
            return 0;
        const int f = first_layer[k];
        return f < 0 ? 0 : (f > L ? L : f);
    }
};

// Solving with a fraction of the record (Sec. 3.2 counts O(L T) memory for the matrices): a
// first pass over all layers keeps only every `stride`-th row of D (checkpoints) and finds the
// final time; then, from the last block of `stride` layers to the first, the block's rows are
// filled again from the checkpoint below it into a small block record and walked back.
//   pass 0 (checkpoints): layers [0, L); row l is kept at slot (l + 1) / stride - 1 when
//                         (l + 1) is a multiple of stride and l + 1 < L
//   pass 1 (one block)  : layers [begin, end), starting from checkpoint slot begin / stride - 1
//                         (from scratch when begin = 0); row l is kept at slot l - begin of the
//                         block record; no final argmin
struct Blocks {
    int pass;
    int begin, end;
    int stride;
    int slots;                    // checkpoint rows per candidate
    float *ckpt;                  // [K][slots][pitch]
    float *block;                 // [K][stride][pitch]
};

struct LevelEntry {   // one visited level of one layer of one candidate
    int32_t shift;    // tau - m_l (INT32_MAX in padding entries)
    float err;
    unsigned long long keep = ~0ull;   // wave-uniform: which of the first 64 entries to visit
};

// The prepare kernel's tables of one layer (see prepare_order).
struct LayerTable {
    const int32_t *shift;   // [s8]
    const int32_t *order;   // [s8]
    const int32_t *start;   // [s8 + kBatch], D record only
    const int32_t *entry;   // [s8], D record only
    int limit;              // a larger shift than this (the reduced budget) is never usable
    // An entry beyond the budget could still "apply" to the padding buckets at the end of a row;
    // it is taken out here, so that every shift the sweep uses is at most the layer's largest
    // usable one (the staged tiles of the global-row path size their window by that).
    __device__ __forceinline__ int32_t usable(int32_t shift) const
    {
        return shift > limit ? INT32_MAX : shift;
    }
};
struct LevelTables {
    const int32_t *shifts, *order, *start, *entry;
    int s8;
    int limit = INT32_MAX;  // set by the fill once it knows the reduced budget
    __device__ __forceinline__ LayerTable layer(int l) const
    {
        return LayerTable{shifts + (size_t)l * s8, order + (size_t)l * s8,
                          start + (size_t)l * (s8 + kBatch), entry + (size_t)l * s8, limit};
    }
};

// This lane's entry of the 64 visited entries of a layer starting at entry `blk`.  With the D
// record an entry stands for all levels of one shift and carries the smallest of their errors.
template <bool kLevel>
__device__ __forceinline__ LevelEntry load_level(LayerTable tl, ErrRow er, int s8, int blk,
                                                 int lane)
{
    LevelEntry p;
    p.shift = INT32_MAX;
    p.err = __builtin_inff();
    const int r = blk + lane;
    if (r < s8) {
        p.shift = tl.usable(tl.shift[r]);
        if constexpr (kLevel) {
            p.err = er.at(tl.order[r]);
        } else {
            const int end = tl.start[r + 1];
            for (int j = tl.start[r]; j < end; ++j) {
                const float e = er.at(tl.order[j]);
                p.err = e < p.err ? e : p.err;
            }
        }
    }
    return p;
}

// Layers of at most 64 levels (one lane per level): what a wave loads for the NEXT layer while
// it sweeps a layer.  No load depends on another, so all are in flight during the sweep.
//   shift : shift of entry `lane` (every wave)
//   raw   : error of level `lane`; with the level record entry r is level r and this is the
//           entry's error; with the D record only the first wave of a team loads it, with
//   entry : the entry level `lane` belongs to, and folds the errors of a team's candidate into
//           the team's table in LDS with one atomic min per lane (publish_entries).
struct LevelFetch {
    int32_t shift;
    float raw;
    int32_t entry;
};

template <bool kLevel>
__device__ __forceinline__ LevelFetch fetch_levels(LayerTable tl, ErrRow er, int S, int s8,
                                                   int lane, bool producer)
{
    LevelFetch f;
    f.shift = lane < s8 ? tl.usable(tl.shift[lane]) : INT32_MAX;
    f.raw = __builtin_inff();
    f.entry = 0;
    if (lane < S && (kLevel || producer)) {
        f.raw = er.at(lane);
        if constexpr (!kLevel)
            f.entry = tl.entry[lane];
    }
    return f;
}

// Level record: a level need not be visited when an earlier level of the layer takes the same
// time with an error no larger: it reads the same cell of D_{l-1}, a rounded add is monotone in
// the addend, so its value cannot be strictly smaller than the earlier one's and the strict "<"
// never selects it.  Bit r of the result is set when level r has to be visited; one wave.
// `twins`: the levels that have a later level of the same time (from the prepare kernel).
__device__ __forceinline__ unsigned long long levels_to_visit(const LevelFetch &f,
                                                              unsigned long long twins, int lane)
{
    bool skip = false;
    while (twins) {
        const int r = __builtin_ctzll(twins);
        twins &= twins - 1;
        const int shift = __builtin_amdgcn_readlane(f.shift, r);
        const float err = __builtin_bit_cast(
            float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, f.raw), r));
        skip |= lane > r && f.shift == shift && err <= f.raw;
    }
    return __ballot(!skip);
}

__device__ __forceinline__ unsigned long long load_twins(LayerTable tl)
{
    return (unsigned long long)(uint32_t)tl.start[0] |
           ((unsigned long long)(uint32_t)tl.start[1] << 32);
}

// table[r] = shift in units of 1 / `scale` buckets and smallest error among the levels of entry r (+inf for unused
// entries); one wave.
__device__ __forceinline__ void publish_entries(int2 *table, const LevelFetch &f, unsigned scale, int S, int lane)
{
    table[lane] = make_int2((int)((unsigned)f.shift * scale), __builtin_bit_cast(int, __builtin_inff()));
    if (lane < S)
        __hip_atomic_fetch_min(reinterpret_cast<float *>(&table[f.entry].y), f.raw, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_WORKGROUP);
}

// The table words of the next layer that are still being loaded while a layer is swept.  Loads
// and stores retire through one in-order counter, so a wait for these loads placed after the
// record stores of a layer would also wait for those stores; `settle` makes the compiler wait
// for the loads where it is called (right after the sweep, when they have long arrived).
struct Pending {
    const LevelFetch *fetch;
    const LevelEntry *entry;
    __device__ __forceinline__ void settle() const
    {
        asm volatile("" ::"v"(fetch->raw), "v"(fetch->shift), "v"(fetch->entry),
                     "v"(entry->shift), "v"(entry->err));
    }
};

__device__ __forceinline__ float lane_value(float v, int lane)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), lane));
}

#include "dp_core.h"

// One workgroup per candidate (and budget); the first L + 1 workgroups do what dp_prepare does, for
// the launches of the full table that follow and take the candidates this one gives up.  Their code comes
// last (they are marked as unlikely): with it in front a change there moved the solve's loops, which
// wait for instructions as much as for anything, and made calls 1.4 - 3.6 % slower.  (16 bytes of s_nop ahead of
// the solve: 1 - 2 % slower; 32 or 64: no change.)
template <bool kFar>
__global__ __launch_bounds__(kCoreThreads) void dp_core(const int32_t *__restrict__ tau,
                                                        ErrSource src, int K, int L, int S,
                                                        PrepareArgs prep, CoreParams cp,
                                                        int16_t *__restrict__ profile,
                                                        float *__restrict__ cost)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char core_lds[];
    __shared__ CoreShared sh;
    if (__builtin_expect((int)blockIdx.x <= L, 0)) {
        prepare(tau, K, L, S, prep, blockIdx.x);
        return;
    }
    const int solve = (int)blockIdx.x - (L + 1);  // candidate k under budget j
    const int j = solve / K, k = solve - j * K;
    const size_t rows = kFar ? 2 * (size_t)cp.far * sizeof(float) : 0;
    solve_core<kFar>(tau, src.of_candidate(k, L, S), L, S, cp.budget[j], cp,
                     cp.spill + (size_t)solve * (rows + cp.spill_bytes) + rows, core_lds, sh,
                     profile + (size_t)solve * L, cost + solve);
}

// Whether the launches of the full table have to solve candidate k: every one, or (behind
// dp_core) those it gave up under any of the `budgets` it tried.
struct Todo {
    const int16_t *profile = nullptr;   // [budgets][K][L]
    int budgets = 0;
    __device__ __forceinline__ bool has(int k, int K, int L) const
    {
        if (!profile)
            return true;
        bool any = false;
        for (int j = 0; j < budgets; ++j)
            any |= profile[((size_t)j * K + k) * L] == kGivenUp;
        return any;
    }
    // the same where k is the same in the whole wave, as a scalar: a row's plan depends on it, and a
    // divergent plan would put the sweep under execution masks
    __device__ __forceinline__ bool has_wave(int k, int K, int L) const
    {
        return !profile || __builtin_amdgcn_readfirstlane(has(k, K, L) ? 1 : 0) != 0;
    }
};

// The levels of one layer swept over one group of R chunks (R*64 consecutive reduced buckets
// from t0); best[j] / arg[j] belong to bucket t0 + 64*j + lane.
//   prev  : row of the previous layer, prev[-kHalo .. -1] reads +inf
//   first : lane i holds visited entry i of the layer (entries 0..63)
//   tl / er : the layer's tables, for entries >= 64
// A level applies to the group if its shift does not exceed the group's last bucket; lanes
// left of the shift then read the +inf apron.  The applicable levels of a 64-block are found
// with one ballot and walked in ascending position.
template <int R, bool kLevel, bool kPairs>
__device__ __forceinline__ void sweep_group(const float *__restrict__ prev, LevelEntry first,
                                            LayerTable tl, ErrRow er, int s8, int t0, int lane,
                                            float (&best)[R], unsigned (&arg)[R])
{
#pragma unroll
    for (int j = 0; j < R; ++j) {
        best[j] = __builtin_inff();
        arg[j] = kNoLevel;
    }
    const int last = t0 + R * kWave - 1;      // last bucket of the group
    __builtin_amdgcn_s_waitcnt(0xC07F);       // lgkmcnt(0): see fill_group_quads
    const char *pl = reinterpret_cast<const char *>(prev + t0 + lane);
    auto row_at = [&](int shift) {
        return reinterpret_cast<const float *>(pl - (size_t)(unsigned)shift * 4u);
    };

    // (with S <= 64 this loop runs once; telling the compiler so made the code slower)
    for (int blk = 0; blk < s8; blk += kWave) {
        const LevelEntry mine =
            blk == 0 ? first : load_level<kLevel>(tl, er, s8, blk, lane);
        unsigned long long use = __ballot(mine.shift <= last);
        if (blk == 0)
            use &= first.keep;
        if constexpr (kLevel) {
            // Two levels (in index order) share one comparison: where the smaller of the two is below
            // what came before, the cell notes the pair, and which of the two it was is found out
            // once at the end.  Strict "<" decides; the value is the min either way (the sign of
            // a zero may differ from a select's, the walk back re-sums the cost).  Add, compare, select
            // and min for every level, 4 operations, are 2.5 for half of a pair: K = 1001, L = 52,
            // S = 42, B = 9973: 1533 us a solve and 1312.  (Comparing once for four levels saves no
            // more: three of them have to be looked at again at the end.)
            auto take_pair = [&](int &p0, int &p1, float &e0, float &e1) __attribute__((always_inline)) {
                const int i0 = __builtin_ctzll(use);
                use &= use - 1;
                const int i1 = __builtin_ctzll(use);
                use &= use - 1;
                p0 = __builtin_amdgcn_readlane(mine.shift, i0);
                p1 = __builtin_amdgcn_readlane(mine.shift, i1);
                e0 = lane_value(mine.err, i0);
                e1 = lane_value(mine.err, i1);
                return (unsigned)(blk + i0) | (unsigned)(blk + i1) << 8;   // (>= 256: i1 > 0)
            };
            int n_use = kPairs ? __builtin_popcountll(use) : 0;
            const bool noted = n_use >= 2;
            for (; n_use >= 4; n_use -= 4) {      // two pairs a trip, so that no minimum is moved
                int sa, sb, sc, sd;
                float ea, eb, ec, ed;
                const unsigned ab = take_pair(sa, sb, ea, eb), cd = take_pair(sc, sd, ec, ed);
                const float *const pa = row_at(sa), *const pb = row_at(sb);
                const float *const pc = row_at(sc), *const pd = row_at(sd);
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const float m = min3(best[j], pa[j * kWave] + ea, pb[j * kWave] + eb);
                    arg[j] = m < best[j] ? ab : arg[j];
                    best[j] = min3(m, pc[j * kWave] + ec, pd[j * kWave] + ed);
                    arg[j] = best[j] < m ? cd : arg[j];
                }
            }
            if (n_use >= 2) {
                int sa, sb;
                float ea, eb;
                const unsigned ab = take_pair(sa, sb, ea, eb);
                const float *const pa = row_at(sa), *const pb = row_at(sb);
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const float m = min3(best[j], pa[j * kWave] + ea, pb[j * kWave] + eb);
                    arg[j] = m < best[j] ? ab : arg[j];
                    best[j] = m;
                }
            }
            while (use) {
                const int i = __builtin_ctzll(use);
                use &= use - 1;
                const float *p = row_at(__builtin_amdgcn_readlane(mine.shift, i));
                const float e = lane_value(mine.err, i);
                const unsigned s = (unsigned)(blk + i);   // visiting order = level index here
#pragma unroll
                for (int j = 0; j < R; ++j) {
                    const float v = p[j * kWave] + e;
                    arg[j] = v < best[j] ? s : arg[j];
                    vmin(best[j], v);
                }
            }
            // the first of a noted pair if it gives the cell's value, otherwise the second (what a
            // later single level beat is below 256 and stays)
#pragma unroll
            for (int j = 0; noted && j < R; ++j) {
                const bool pair = arg[j] > kNoLevel;
                const int i = (int)(arg[j] & 0xFF) - blk;
                const int shift = __builtin_amdgcn_ds_bpermute(4 * i, mine.shift);
                const float e = __builtin_bit_cast(
                    float, __builtin_amdgcn_ds_bpermute(4 * i, __builtin_bit_cast(int, mine.err)));
                const float v = row_at(pair ? shift : 0)[j * kWave] + e;
                const unsigned s = v == best[j] ? arg[j] & 0xFF : arg[j] >> 8;
                arg[j] = pair ? s : arg[j];
            }
        } else {
            // sorted by shift: the applicable levels are the first n_use of the block
            const int n_use = __builtin_popcountll(use);
            int i = 0;
            for (; i + 2 <= n_use; i += 2) {
                const float *p0 = row_at(__builtin_amdgcn_readlane(mine.shift, i));
                const float *p1 = row_at(__builtin_amdgcn_readlane(mine.shift, i + 1));
                const float e0 = lane_value(mine.err, i);
                const float e1 = lane_value(mine.err, i + 1);
#pragma unroll
                for (int j = 0; j < R; ++j)
                    vmin3(best[j], p0[j * kWave] + e0, p1[j * kWave] + e1);
            }
            if (i < n_use) {
                const float *p0 = row_at(__builtin_amdgcn_readlane(mine.shift, i));
                const float e0 = lane_value(mine.err, i);
#pragma unroll
                for (int j = 0; j < R; ++j)
                    vmin(best[j], p0[j * kWave] + e0);
            }
            if (n_use < kWave)
                break;                        // later blocks only hold larger shifts
        }
    }
}

// ---------------------------------------------------------------------------------------------
// The D-record sweep with 128-bit LDS reads (layers of at most 64 levels).  Aligned 128-bit reads
// move twice the bytes per clock of narrower ones, so a lane takes four consecutive buckets:
//   * the first 252 Q buckets of a wave's group are Q "quad chunks": lane i >= 1 owns buckets
//     252 j + 4 (i - 1) .. + 3 of quad chunk j, and one read gives it the four values
//     row[4 q .. 4 q + 3] of the aligned quad q = (its own quad) - (shift / 4);
//   * for a shift that is not a multiple of four these are the values of four buckets that begin
//     (shift mod 4) further on: the entries of a layer are visited by that residue (the prepare
//     kernel orders them), and the minima move by a bucket from one to the next (sweep_layer).
//     Lane 0 has no bucket of its own: it reads the quad below lane 1's and only serves as left
//     neighbour of that move (63 of 64 lanes work);
//   * the remaining buckets of the group, fewer than 252, are covered by T ordinary chunks of 64
//     (32-bit reads, lane = bucket) placed at the END of the group; they may overlap the quad
//     chunks by up to 63 buckets, which are then computed twice with the same result.
// R chunks of 64 thus become Q quad chunks and T tail chunks, 4 Q + T <= R + 1 registers.
typedef float float4v __attribute__((ext_vector_type(4)));

// x of the lane to the left (lane 0 gets 0.0f, which nothing uses)
__device__ __forceinline__ float from_left(float x)
{
    return __int_as_float(
        __builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x138 /* wave_shr:1 */, 0xf, 0xf, true));
}

// Two entries of a table in LDS (shift, error, and again), one read wherever the first of them lies.
// Shifts are in bytes, but in buckets where a row is read from memory (kBuckets): bytes would pass 2^31.
// (Two values of their own the compiler fetches one at a time, the second where it is needed.)
typedef int EntryPair __attribute__((ext_vector_type(4), aligned(8)));

// The entries of one residue that a group can use: `n` consecutive ones from `at` on, of which the
// first two are here already.
struct EntryRun {
    const int2 *at;
    int n;
    EntryPair pair;
};
__device__ __forceinline__ EntryPair entry_pair(const int2 *at)
{
    return *reinterpret_cast<const EntryPair *>(at);
}

// kSplit: the waves of a workgroup come in two halves that sweep the same chunks, each visiting
// every other pair of the run's entries (a run's odd last entry counts as a pair); `skip`: the
// run's first pair is the other half's.
template <bool kSplit>
__device__ __forceinline__ EntryRun entry_run(const int2 *entries, unsigned long long use, bool skip)
{
    EntryRun r;
    r.at = entries + (use ? __builtin_ctzll(use) : 0);
    r.n = __builtin_popcountll(use);
    if (kSplit && skip) {
        r.at += 2;
        r.n -= 2;
    }
    r.pair = entry_pair(r.at);
    return r;
}

// bq[j][c] and bt[j] become the least over the run's entries, quads[j] and tail[j] being what an
// entry of shift kRes and 0 reads.  Shifts and errors come from LDS as the same word for every lane, two entries
// at a time and a trip ahead: moved from a lane by v_readlane (and the error back to a vector register)
// they cost 28 clocks of the pipe that the mins need, more than four quads of mins do.  That pipe takes four
// clocks for any instruction but fp32 adds and multiplies of vector registers only, which have a
// second one (v_min3 4.0 clocks of a SIMD, v_add 2.0, v_add with a scalar or a lane to the left 4.0).
// kBatched: all quads of a pair are asked for before the first of them is used.  The compiler does so by itself, but not
// in the loop over blocks of layers of dp_rest, where it runs out of scalar registers and reads a quad at a time.  us a call
// with checkpoints of which eleven candidates are given up, so and batched: K = 1024, L = 54, S = 40, B = 10^4 788 and 697;
// K = 2000, B = 3000 833 and 692.
constexpr int kMaxBatched = 5;       // (more quads at once than that: registers in scratch memory)
template <int Q, int T, int kRes, bool kSplit, bool kBuckets, bool kBatched>
__device__ __forceinline__ void sweep_run(const float4v *quads, const float *tail,
                                          EntryRun run, float (&bq)[Q > 0 ? Q : 1][4], float (&bt)[T > 0 ? T : 1])
{
    constexpr int kStep = kSplit ? 4 : 2;
    using Shift = std::conditional_t<kBuckets, ptrdiff_t, int>;
    constexpr Shift kBytes = kBuckets ? 4 : 1;    // of a unit
    auto quads_at = [&](Shift shift) {
        return reinterpret_cast<const float4v *>(reinterpret_cast<const char *>(quads) - shift * kBytes +
                                                 4 * kRes);
    };
    auto tail_at = [&](Shift shift) {
        return reinterpret_cast<const float *>(reinterpret_cast<const char *>(tail) - shift * kBytes);
    };
    for (; run.n >= 2; run.n -= kStep) {
        const EntryPair now = run.pair;
        run.at += kStep;
        run.pair = entry_pair(run.at);
        const float e0 = __int_as_float(now.y), e1 = __int_as_float(now.w);
        if constexpr (Q > 0) {
            const float4v *q0 = quads_at(now.x), *q1 = quads_at(now.z);
            if constexpr (kBatched) {
                constexpr int kAtOnce = Q <= kMaxBatched ? Q : (Q + 1) / 2;
#pragma unroll
                for (int j0 = 0; j0 < Q; j0 += kAtOnce) {
                    float4v v0[kAtOnce], v1[kAtOnce];
#pragma unroll
                    for (int j = 0; j < kAtOnce && j0 + j < Q; ++j) {
                        v0[j] = q0[(j0 + j) * kQuadLanes];
                        v1[j] = q1[(j0 + j) * kQuadLanes];
                    }
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int j = 0; j < kAtOnce && j0 + j < Q; ++j)
#pragma unroll
                        for (int c = 0; c < 4; ++c)
                            vmin3(bq[j0 + j][c], v0[j][c] + e0, v1[j][c] + e1);
                }
            } else {
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    const float4v v0 = q0[j * kQuadLanes], v1 = q1[j * kQuadLanes];
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        vmin3(bq[j][c], v0[c] + e0, v1[c] + e1);
                }
            }
        }
        if constexpr (T > 0) {
            const float *p0 = tail_at(now.x), *p1 = tail_at(now.z);
#pragma unroll
            for (int j = 0; j < T; ++j)
                vmin3(bt[j], p0[j * kWave] + e0, p1[j * kWave] + e1);
        }
    }
    if (run.n == 1) {
        const float e = __int_as_float(run.pair.y);
        if constexpr (Q > 0) {
            const float4v *q = quads_at(run.pair.x);
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                const float4v v = q[j * kQuadLanes];
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    vmin(bq[j][c], v[c] + e);
            }
        }
        if constexpr (T > 0) {
            const float *p = tail_at(run.pair.x);
#pragma unroll
            for (int j = 0; j < T; ++j)
                vmin(bt[j], p[j * kWave] + e);
        }
    }
}

// The same for all entries of a layer (`shift`: that of entry `lane`) over a group of ordinary chunks alone, where
// residues do not matter.  Few cells of few levels would wait for a round trip to LDS per residue, and another for
// the entries: here shifts come from lanes, four entries a trip, and the errors arrive beside the cells.  An
// entry that the group cannot use reads the cell itself and adds +inf.
template <int T>
__device__ __forceinline__ void sweep_tails(const float *tail, const int2 *entries, int shift,
                                            int last_bucket, int lane, float (&bt)[T])
{
    float err = __int_as_float(entries[lane].y);
    const bool use = shift <= last_bucket;
    const int usable = use ? shift * (int)sizeof(float) : 0;
    const int n = kWave - __builtin_clzll(__ballot(use) | 1);
    for (int i = 0; i < n; i += 4) {
        const float *p[4];
        float v[4][T];
#pragma unroll
        for (int q = 0; q < 4; ++q)
            p[q] = reinterpret_cast<const float *>(reinterpret_cast<const char *>(tail) -
                                                   __builtin_amdgcn_readlane(usable, i + q));
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int j = 0; j < T; ++j)
                v[q][j] = p[q][j * kWave];
        if (i == 0)
            err = use ? err : __builtin_inff();
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
            const float e0 = lane_value(err, i + q), e1 = lane_value(err, i + q + 1);
#pragma unroll
            for (int j = 0; j < T; ++j)
                vmin3(bt[j], v[q][j] + e0, v[q + 1][j] + e1);
        }
    }
}

// All entries of a layer (at most 64, `mine.shift`: that of entry `lane`) over one group.  An entry of
// residue r adds to the whole quads it reads, four buckets from 4 q + r on; so the minima are kept shifted by
// the residue, and moved by one bucket (which is a move of a fourth of them to the lane to the right,
// the others only change their names) from one residue to the next, 3 to 0.  An operand from the left
// lane in every add, as before, took the slow pipe.  What lane 0 gets from the left ends in buckets that are not
// its own and never reaches lane 1.
// kAhead: the first entries of all four runs are asked for at once (registers permitting).
template <int Q, int T, bool kSplit, bool kAhead, bool kBuckets, bool kBatched = false>
__device__ __forceinline__ void sweep_layer(const float4v *quads, const float *tail,
                                            const int2 *entries, LevelEntry mine, int last_bucket,
                                            int half, float (&bq)[Q > 0 ? Q : 1][4],
                                            float (&bt)[T > 0 ? T : 1])
{
    const unsigned long long use = __ballot(mine.shift <= last_bucket);
    const int residue = mine.shift & 3;
    const unsigned long long use0 = use & __ballot(residue == 0);
    const unsigned long long use1 = use & __ballot(residue == 1);
    const unsigned long long use2 = use & __ballot(residue == 2);
    const unsigned long long use3 = use & __ballot(residue == 3);
    // Scalar loads and LDS reads share one counter, and scalar loads return out of order: while
    // one is in flight (the wall clock of the priority turns, the next layer's chunk range)
    // every wait for an LDS read in the sweep has to be a wait for ALL of them, and a wave
    // cannot start on the first quads while the later ones arrive.  Let them land first.
    __builtin_amdgcn_s_waitcnt(0xC07F);           // lgkmcnt(0), nothing else
    // kSplit: the pairs of entries are numbered through the four runs; half h visits the
    // pairs whose number is h mod 2, so both halves get every residue's kind of work
    int turn = half;
    auto pairs = [](unsigned long long u) { return (__builtin_popcountll(u) + 1) >> 1; };
    EntryRun run3 = entry_run<kSplit>(entries, use3, turn & 1);
    turn += kSplit ? pairs(use3) : 0;
    EntryRun run2 = entry_run<kSplit>(entries, use2, turn & 1);
    turn += kSplit ? pairs(use2) : 0;
    EntryRun run1 = entry_run<kSplit>(entries, use1, turn & 1);
    turn += kSplit ? pairs(use1) : 0;
    EntryRun run0 = entry_run<kSplit>(entries, use0, turn & 1);
    auto later = [](EntryRun &r) __attribute__((always_inline)) {
        if (!kAhead) {
            asm volatile("" ::: "memory");
            r.pair = entry_pair(r.at);
        }
    };
    auto next_residue = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const float carry = from_left(bq[j][3]);
            bq[j][3] = bq[j][2];
            bq[j][2] = bq[j][1];
            bq[j][1] = bq[j][0];
            bq[j][0] = carry;
        }
    };
    sweep_run<Q, T, 3, kSplit, kBuckets, kBatched>(quads, tail, run3, bq, bt);
    next_residue();
    later(run2);
    sweep_run<Q, T, 2, kSplit, kBuckets, kBatched>(quads, tail, run2, bq, bt);
    next_residue();
    later(run1);
    sweep_run<Q, T, 1, kSplit, kBuckets, kBatched>(quads, tail, run1, bq, bt);
    next_residue();
    later(run0);
    sweep_run<Q, T, 0, kSplit, kBuckets, kBatched>(quads, tail, run0, bq, bt);
}

// One group of one layer (D record, at most 64 levels), Q quad chunks and T ordinary ones from bucket
// `tail0` of the group on: sweep with 128-bit reads, store the record, write the new row values; the barrier
// protocol is fill_group's.
// prev + t0 is 16-byte aligned (rows, aprons and chunk starts are multiples of four floats).
// kSplit (in place only): this wave has a twin in the other half of the workgroup with the same
// group; the two visit alternate pairs of the layer's entries, the second half (`half` = 1)
// leaves its minima in `part` (indexed like the row) before the barrier, and the first half
// folds them into its own behind it.  min is exact and order-blind here, so the row is the one
// a single wave would have computed.
// kTails: sweep_tails does it.
template <int Q, int T, int tail0, bool inplace, bool kSplit, bool kAhead, bool kBuckets, bool kBatched,
          bool kTails = false>
__device__ __forceinline__ void fill_group_quads(const float *prev, float *cur, float *rec,
                                                 LevelEntry first, const int2 *entries, int t0,
                                                 int lane, Pending pending, int half, float *part)
{
    static_assert(!kSplit || inplace, "the halves meet at the in-place barrier");
    static_assert(!kTails || (Q == 0 && !kSplit && !kBuckets), "ordinary chunks of a row in LDS");
    if constexpr (Q + T == 0) {
        pending.settle();
        if (inplace)
            __syncthreads();
    } else {
        float bq[Q > 0 ? Q : 1][4], bt[T > 0 ? T : 1];
#pragma unroll
        for (int j = 0; j < Q; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                bq[j][c] = __builtin_inff();
#pragma unroll
        for (int j = 0; j < T; ++j)
            bt[j] = __builtin_inff();
        // last bucket of the group
        const int last = t0 + (T > 0 ? tail0 + T * kWave : Q * kQuadChunk) - 1;
        const float4v *quads = reinterpret_cast<const float4v *>(prev + t0) + (lane - 1);
        const float *tail = prev + t0 + tail0 + lane;
        if constexpr (kTails)
            sweep_tails<T>(tail, entries, first.shift, last, lane, bt);
        else
            sweep_layer<Q, T, kSplit, kAhead, kBuckets, kBatched>(quads, tail, entries, first, last, half, bq, bt);
        pending.settle();
        const int tq = t0 + 4 * (lane - 1);       // this lane's first bucket of quad chunk 0
        const int tt = t0 + tail0 + lane;
        if constexpr (kSplit) {
            if (half) {
                if (lane > 0) {
#pragma unroll
                    for (int j = 0; j < Q; ++j) {
                        const float4v v = {bq[j][0], bq[j][1], bq[j][2], bq[j][3]};
                        *reinterpret_cast<float4v *>(part + tq + j * kQuadChunk) = v;
                    }
                }
#pragma unroll
                for (int j = 0; j < T; ++j)
                    part[tt + j * kWave] = bt[j];
            }
            __syncthreads();                      // every read of the row is done, `part` is written
            if (half)
                return;
            if (lane > 0) {
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    const float4v v = *reinterpret_cast<const float4v *>(part + tq + j * kQuadChunk);
                    vmin(bq[j][0], v.x);
                    vmin(bq[j][1], v.y);
                    vmin(bq[j][2], v.z);
                    vmin(bq[j][3], v.w);
                }
            }
#pragma unroll
            for (int j = 0; j < T; ++j)
                vmin(bt[j], part[tt + j * kWave]);
        }
        if (rec) {       // streamed: the record is not read again before the walk back
            if (lane > 0) {
#pragma unroll
                for (int j = 0; j < Q; ++j) {
                    const float4v v = {bq[j][0], bq[j][1], bq[j][2], bq[j][3]};
                    __builtin_nontemporal_store(
                        v, reinterpret_cast<float4v *>(rec + tq + j * kQuadChunk));
                }
            }
#pragma unroll
            for (int j = 0; j < T; ++j)
                __builtin_nontemporal_store(bt[j], &rec[tt + j * kWave]);
        }
        if (inplace && !kSplit)
            __syncthreads();
        if (lane > 0) {
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                const float4v v = {bq[j][0], bq[j][1], bq[j][2], bq[j][3]};
                *reinterpret_cast<float4v *>(cur + tq + j * kQuadChunk) = v;
            }
        }
#pragma unroll
        for (int j = 0; j < T; ++j)
            cur[tt + j * kWave] = bt[j];
    }
}

// One group of one layer: sweep, store the record, and write the new row values to `cur`.
// With `inplace` cur aliases prev, so a workgroup barrier separates the last read of the row
// from the first write (every wave of the workgroup calls this exactly once per layer then,
// with R = 0 if it has no chunks).
template <int R, bool kLevel, bool inplace, bool kPairs>
__device__ __forceinline__ void fill_group(const float *prev, float *cur, uint8_t *choice,
                                           float *rec, LevelEntry first, LayerTable tl, ErrRow er,
                                           int s8, int t0, int lane, Pending pending)
{
    if constexpr (R == 0) {
        pending.settle();
        if (inplace)
            __syncthreads();
    } else {
        float best[R];
        unsigned arg[R];
        sweep_group<R, kLevel, kPairs>(prev, first, tl, er, s8, t0, lane, best, arg);
        pending.settle();
        const int tl = t0 + lane;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if constexpr (kLevel)
                choice[tl + j * kWave] = (uint8_t)arg[j];
            else if (rec)   // streamed: the record is not read again before the walk back
                __builtin_nontemporal_store(best[j], &rec[tl + j * kWave]);
        }
        if (inplace)
            __syncthreads();
#pragma unroll
        for (int j = 0; j < R; ++j)
            cur[tl + j * kWave] = best[j];
    }
}

template <bool kLevel, bool inplace, int kMax, bool kQuads, bool kSplit, bool kAhead, bool kBuckets, bool kPairs,
          bool kBatched>
__device__ __forceinline__ void fill_group_n(int r, const float *prev, float *cur, uint8_t *choice,
                                             float *rec, LevelEntry first, const int2 *entries,
                                             LayerTable tl, ErrRow er, int s8, int t0, int lane,
                                             Pending pending, int half = 0, float *part = nullptr)
{
    static_assert(!kSplit || kQuads, "only the 128-bit sweep splits a layer's entries");
    switch (r) {
#define SPDY_CASE(RR)                                                                          \
    case RR:                                                                                   \
        if constexpr (RR <= kMax) {                                                            \
            if constexpr (kQuads)                                                              \
                fill_group_quads<quad_chunks(RR), tail_chunks(RR), (RR - tail_chunks(RR)) * kWave, \
                                 inplace, kSplit, kAhead, kBuckets, kBatched>(                 \
                    prev, cur, rec, first, entries, t0, lane, pending, half, part);            \
            else                                                                               \
                fill_group<RR, kLevel, inplace, kPairs>(prev, cur, choice, rec, first, tl, er, s8, t0, \
                                                lane, pending);                                \
        }                                                                                      \
        break;
        SPDY_CASE(0)
        SPDY_CASE(1)
        SPDY_CASE(2)
        SPDY_CASE(3)
        SPDY_CASE(4)
        SPDY_CASE(5)
        SPDY_CASE(6)
        SPDY_CASE(7)
        SPDY_CASE(8)
        SPDY_CASE(9)
        SPDY_CASE(10)
        SPDY_CASE(11)
        SPDY_CASE(12)
        SPDY_CASE(13)
        SPDY_CASE(14)
        SPDY_CASE(15)
        SPDY_CASE(16)
        SPDY_CASE(17)
        SPDY_CASE(18)
        SPDY_CASE(19)
        SPDY_CASE(20)
        SPDY_CASE(21)
        SPDY_CASE(22)
        SPDY_CASE(23)
        SPDY_CASE(24)
        SPDY_CASE(25)
        SPDY_CASE(26)
        SPDY_CASE(27)
        SPDY_CASE(28)
#undef SPDY_CASE
    }
}

// The same in place for a share of whole quad chunks, or (kTails) of ordinary ones.
template <bool kTails, bool kBatched>
__device__ __forceinline__ void fill_share_n(int share, float *row, float *rec, LevelEntry first,
                                             const int2 *entries, int lane, Pending pending)
{
    const int t0 = (share & 0xFFFFF) * 4;
    switch (share >> 20 & 0xF) {
#define SPDY_CASE(NN)                                                                          \
    case NN:                                                                                   \
        if constexpr (NN <= kMaxQuads)                                                         \
            fill_group_quads<NN, 0, 0, true, false, true, false, kBatched>(                    \
                row, row, rec, first, entries, t0, lane, pending, 0, nullptr);                 \
        else if constexpr (kTails)                                                             \
            fill_group_quads<0, NN - kMaxQuads, 0, true, false, false, false, kBatched, true>( \
                row, row, rec, first, entries, t0, lane, pending, 0, nullptr);                 \
        break;
        SPDY_CASE(0)
        SPDY_CASE(1)
        SPDY_CASE(2)
        SPDY_CASE(3)
        SPDY_CASE(4)
        SPDY_CASE(5)
        SPDY_CASE(6)
        SPDY_CASE(7)
        SPDY_CASE(8)
        SPDY_CASE(9)
        SPDY_CASE(10)
        SPDY_CASE(11)
        SPDY_CASE(12)
        SPDY_CASE(13)
#undef SPDY_CASE
    }
    static_assert(kMaxQuads + kFewChunks == 13, "a case for each");
}

// (value, t) pairs ordered by value, then by smaller t.
__device__ __forceinline__ void argmin_merge(float &bv, int &bt, float v, int t)
{
    if (v < bv || (v == bv && t < bt)) {
        bv = v;
        bt = t;
    }
}

// kNoCost: `cost` may be nullptr, the time is all that the caller asked for.
template <bool kNoCost>
__device__ __forceinline__ void write_result(float bv, int bt, int k, int32_t *tstar, float *cost)
{
    if (!kNoCost || cost)
        cost[k] = bv;
    tstar[k] = (bv < __builtin_inff()) ? bt : -1;   // -1: no profile meets the budget
}

#include "dp_small.h"
#include "dp_columns.h"

// ---------------------------------------------------------------------------------------------
// Walk back through the D record: one wave per candidate.  At (l, t) the lanes try the levels in parallel: lane s
// forms D_{l-1}[t - shift_s] + err[l][s] with the same single fp32 add as the fill and compares
// it with D_l[t]; the lowest matching level is the one a strict "<" sweep would have kept.
// Only the gather of D_{l-1} depends on t, so it is issued first and the shifts and errors of the
// next layer down are fetched behind it: one memory round trip per layer on the critical path.
// The cost is then re-summed over the profile in layer order, which reproduces the sign of a
// zero exactly as the level-tracking sweep would (min(+0, -0) is order-blind).
// kLevelBlocks: 64-level blocks a lane holds (1 for S <= 64, 4 for S <= 255).
template <int kLevelBlocks>
struct LayerLevels {
    int shift[kLevelBlocks];      // tau[l][s] - m_l for s = 64 b + lane (INT32_MAX past S)
    float err[kLevelBlocks];
    int reach;                    // computed buckets of row l - 1 (1 for l = 0: only t = 0)
};

template <int kLevelBlocks>
__device__ __forceinline__ LayerLevels<kLevelBlocks> load_layer(
    const int32_t *__restrict__ tau, ErrRow er, const int32_t *__restrict__ meta, int l, int L,
    int S, int lane)
{
    LayerLevels<kLevelBlocks> v;
    const int m = meta[kMetaHeader + l];
    v.reach = l > 0 ? meta[kMetaHeader + L + l - 1] * kWave : 1;
#pragma unroll
    for (int b = 0; b < kLevelBlocks; ++b) {
        const int s = b * kWave + lane;
        v.shift[b] = INT32_MAX;
        v.err[b] = __builtin_inff();
        if (s < S) {
            v.shift[b] = tau[(size_t)l * S + s] - m;
            v.err[b] = er.at(s);
        }
    }
    return v;
}

// One wave walks candidate k back through layers [lb, le) from time t, which it returns as it is
// below layer lb (-1: no profile meets the budget; -2: a damaged record).  row_of(l): row of layer l.
template <int kLevelBlocks, class RowOf>
__device__ __forceinline__ int walk_layers(const int32_t *__restrict__ tau, const ErrSource src,
                                           const int32_t *__restrict__ meta, RowOf row_of, int t,
                                           int lb, int le, int L, int S,
                                           int16_t *__restrict__ prof)
{
    const int lane = threadIdx.x & (kWave - 1);
    if (t < 0) {
        for (int l = lb + lane; l < le; l += kWave)
            prof[l] = t == -1 ? -1 : -2;         // -1: no profile meets the budget
        return t;
    }
    float target = row_of(le - 1)[t];
    LayerLevels<kLevelBlocks> next =
        load_layer<kLevelBlocks>(tau, src.layer(le - 1, S), meta, le - 1, L, S, lane);
    for (int l = le - 1; l >= lb; --l) {
        const LayerLevels<kLevelBlocks> cur = next;
        const float *prow = row_of(l > 0 ? l - 1 : 0);       // row of layer l - 1
        // issue the gather of D_{l-1} first, then the next layer's table behind it
        int u[kLevelBlocks];
        float pv[kLevelBlocks];
        bool valid[kLevelBlocks];
#pragma unroll
        for (int b = 0; b < kLevelBlocks; ++b) {
            const long long uu = (long long)t - cur.shift[b];
            valid[b] = b * kWave < S && uu >= 0 && uu < cur.reach;
            u[b] = valid[b] ? (int)uu : 0;
            pv[b] = __builtin_inff();
            if (valid[b])
                pv[b] = l > 0 ? __builtin_nontemporal_load(&prow[u[b]]) : -0.0f;
        }
        if (l > lb)
            next = load_layer<kLevelBlocks>(tau, src.layer(l - 1, S), meta, l - 1, L, S, lane);
        int found = -1, next_t = 0;
        float next_target = 0.0f;
#pragma unroll
        for (int b = 0; b < kLevelBlocks; ++b) {
            if (b * kWave < S && found < 0) {
                const bool match = valid[b] && pv[b] + cur.err[b] == target;
                const unsigned long long mask = __ballot(match);
                if (mask) {
                    const int first = __builtin_ctzll(mask);
                    found = b * kWave + first;
                    next_t = __shfl(u[b], first, kWave);
                    next_target = __shfl(pv[b], first, kWave);
                }
            }
        }
        if (found < 0) {     // cannot happen on a filled record
            for (int i = lane; i < L; i += kWave)
                prof[i] = -2;
            return -2;
        }
        if (lane == 0)
            prof[l] = (int16_t)found;
        t = next_t;
        target = next_target;
    }
    return t;
}

// ---------------------------------------------------------------------------------------
// The same for all layers of at most 64 levels by a guess of the path.  A walk that gathers a layer's entries of
// the row below and then knows where the next layer's are waits for memory once per layer, 0.97 us with a
// thousand candidates.  Which level the next layers take is nearly always known before, though: on a path of
// least cost all layers trade cost for time at about the same price, the slope of the last row at its final time,
// and take the level of least error + price * shift.  So the entries of up to kGuessed layers are asked for at once,
// each where the guesses above it lead; then the layers are decided as ever, by comparing their entries, and
// where one takes another shift than was guessed, those below are asked for again.  A guess only says what is read
// ahead, never what is taken.
// Of a layer's entries, those beyond the guessed level by more than kGuessSlack are only asked for where none
// before them fits: the least level that fits counts.  Where guesses fail, fewer layers are asked for at once.
// What bounds it: a trip to memory a block, and as long again for the instructions of a wave by itself.  us a
// walk, L = 54, S = 40, B = 10^4, a layer a trip and so: K = 300 51.8 and 34.3, K = 1024 54.6 and 37.5, K = 2048
// 71.4 and 42.4, K = 4096 87.4 and 57.4; L = 200, S = 64, B = 3000, K = 600 202 and 94.  (As plain code, with
// branches around every load and scans one after the other, it took 55 at K = 1024 and 118 at K = 4096.)
//   Price: the least fall of the last row per bucket over the 64 samples between 1/200 and 1/8 of the final
//   time below it.  (A row is not quite convex: from the next bucket below on, one of 64 samples is nearly as
//   low as the last one now and then, and every third guess or more is wrong.  1 - 4 of 54 layers are so.)
// ---------------------------------------------------------------------------------------
constexpr int kGuessed = 8, kGuessSlack = 4, kGuessLayers = 48, kGuessWaves = 16;

struct GuessedLayers {           // of layers top, top - 1, ...; below the first one, the first once more
    int shift[kGuessed];         // of level `lane`; until settle() with what lane j has in `least`
    float err[kGuessed];
    int least, reach;            // of layer top - j in lane j (see LayerLevels)
    __device__ __forceinline__ void load(const int32_t *__restrict__ tau, const ErrSource &src,
                                         const int32_t *__restrict__ meta, int top, int L, int S, int lane)
    {
        const int s = min(lane, S - 1), mine = max(top - (lane & (kGuessed - 1)), 0);
        least = meta[kMetaHeader + mine];
        reach = meta[kMetaHeader + L + max(mine - 1, 0)];
#pragma unroll
        for (int j = 0; j < kGuessed; ++j)
            shift[j] = tau[(size_t)max(top - j, 0) * S + s];
        if (src.err) {
#pragma unroll
            for (int j = 0; j < kGuessed; ++j)
                err[j] = src.err[(size_t)max(top - j, 0) * S + s];
        } else {
            const float w = src.w[s];
#pragma unroll
            for (int j = 0; j < kGuessed; ++j)
                err[j] = __fmul_rn(src.c[max(top - j, 0)], w);
        }
    }
    __device__ __forceinline__ void settle(int top, int S, int lane)
    {
        reach = top - (lane & (kGuessed - 1)) > 0 ? reach * kWave : 1;
#pragma unroll
        for (int j = 0; j < kGuessed; ++j)
            shift[j] = lane < S ? shift[j] - from_lane(least, j) : INT32_MAX;
    }
};

template <class RowOf>
__device__ __forceinline__ int walk_guessed(const int32_t *__restrict__ tau, const ErrSource src,
                                            const int32_t *__restrict__ meta, RowOf row_of, int t, int L, int S,
                                            int16_t *__restrict__ prof)
{
    const int lane = threadIdx.x & (kWave - 1);
    t = uniform(t);
    if (t < 0) {
        for (int l = lane; l < L; l += kWave)
            prof[l] = t == -1 ? -1 : -2;         // (see walk_layers)
        return t;
    }
    GuessedLayers cur, next;
    cur.load(tau, src, meta, L - 1, L, S, lane);
    const float *const last = row_of(L - 1);
    const int back = t / 200 + 1 + lane * max(t >> 9, 1);
    const float below = last[max(t - back, 0)];
    float target = uniform(last[t]);
    float price = back <= t ? (below - target) / (float)back : __builtin_inff();
    price = fminf(from_lane(wave_scan(price, __builtin_inff(), Smaller{}), kWave - 1), 3.4e38f);
    int ahead = kGuessed;                        // layers that are asked for at once
    for (int top = L - 1; top >= 0; top -= kGuessed) {
        cur.settle(top, S, lane);
        // The least score as a word that orders like it, the level in its lowest bits.  (Step by step over all
        // layers: eight chains, not one after the other.)
        unsigned key[kGuessed];
#pragma unroll
        for (int j = 0; j < kGuessed; ++j) {
            const int bits = __float_as_int(__builtin_fmaf(price, (float)cur.shift[j], cur.err[j]));
            const unsigned up = (unsigned)(bits ^ (bits >> 31 | INT32_MIN));
            key[j] = lane < S ? (up & ~63u) | (unsigned)lane : ~0u;
        }
        auto least_of = [&](auto ctrl, auto rows) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < kGuessed; ++j)
                key[j] = min(key[j], dpp_from<decltype(ctrl)::value, decltype(rows)::value>(~0u, key[j]));
            __builtin_amdgcn_sched_barrier(0);
        };
        least_of(Many<0x111>{}, Many<0xf>{});    // (see wave_scan)
        least_of(Many<0x112>{}, Many<0xf>{});
        least_of(Many<0x114>{}, Many<0xf>{});
        least_of(Many<0x118>{}, Many<0xf>{});
        least_of(Many<0x142>{}, Many<0xa>{});
        least_of(Many<0x143>{}, Many<0xc>{});
        int by[kGuessed], near[kGuessed];        // the guessed level's shift; shifts that are asked for
#pragma unroll
        for (int j = 0; j < kGuessed; ++j) {
            const int level = (int)(from_lane(key[j], kWave - 1) & 63u);
            by[j] = from_lane(cur.shift[j], level);
            near[j] = lane <= level + kGuessSlack ? cur.shift[j] : INT32_MAX;
        }
        const int n = min(kGuessed, top + 1);
        int pos = 0, whole = -1;                 // layers that are decided; the one with all levels asked for
        int held = 0;                            // the level of layer top - j, in lane j
        float from[kGuessed] = {};
        do {
            const unsigned want = ((1u << min(n, pos + ahead)) - 1) & ~((1u << pos) - 1);
            int at = t;
#pragma unroll
            for (int j = 0; j < kGuessed; ++j)
                if (want >> j & 1) {
                    // (what is out of reach is not read; rows of a batch are far shorter than 2^29 buckets)
                    const __amdgpu_buffer_rsrc_t row =
                        __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(row_of(max(top - j - 1, 0))), 0,
                                                          from_lane(cur.reach, j) * 4, 0x20000);
                    const unsigned u = min((unsigned)(at - near[j]), 0x3FFFFFFFu);
                    from[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(row, u * 4, 0, 2));
                    at = max(at - by[j], -1);    // (-1: nowhere)
                }
            if (pos == 0 && whole < 0)           // (the first time)
                next.load(tau, src, meta, top - kGuessed, L, S, lane);
            bool as_guessed = true, none = false;
#pragma unroll
            for (int j = 0; j < kGuessed; ++j)
                if (as_guessed && (want >> j & 1)) {
                    const float v = top > j ? from[j] : -0.0f;
                    const unsigned long long fits =
                        __ballot((unsigned)(t - near[j]) < (unsigned)from_lane(cur.reach, j) &&
                                 v + cur.err[j] == target);
                    if (fits) {
                        const int found = __builtin_ctzll(fits), shift = from_lane(cur.shift[j], found);
                        held = lane == j ? found : held;
                        target = from_lane(v, found);
                        t -= shift;
                        as_guessed = shift == by[j];
                        pos = j + 1;
                    } else {
                        as_guessed = false;
                        none = true;
                    }
                }
            ahead = as_guessed ? min(4 * ahead, kGuessed) : (ahead + 1) / 2;
            if (none) {
                if (whole == pos) {              // cannot happen on a filled record
                    for (int i = lane; i < L; i += kWave)
                        prof[i] = -2;
                    return -2;
                }
                whole = pos;
#pragma unroll
                for (int j = 0; j < kGuessed; ++j)
                    near[j] = j == pos ? cur.shift[j] : near[j];
            }
        } while (pos < n);
        if (lane < n)
            prof[top - lane] = (int16_t)held;
        cur = next;
    }
    return t;
}

// The cost of a walked profile, summed in layer order.  Lane 0 wrote the profile; it is made visible
// to the wave first.  Lane i fetches the error of layer 64 b + i (all layers of a block of 64 in one
// round trip instead of one after the other); the sum itself runs over the lanes in order.
__device__ __forceinline__ float profile_cost(const ErrSource src, int L, int S,
                                              const int16_t *__restrict__ prof)
{
    const int lane = threadIdx.x & (kWave - 1);
    __threadfence_block();
    float acc = -0.0f;
    for (int base = 0; base < L; base += kWave) {
        const int l = base + lane;
        float e = 0.0f;
        if (l < L)
            e = src.layer(l, S).at(prof[l]);
        const int n = min(kWave, L - base);
        for (int i = 0; i < n; ++i)
            acc += lane_value(e, i);
    }
    return acc;
}

// ---------------------------------------------------------------------------------------------
// The fill (Eq. 2-3 for all L layers) and the final argmin over t.  The waves of a workgroup
// form `teams` teams of `tw` waves; team i of workgroup b solves candidate b * teams + i.
// Barriers are workgroup-wide, so every team steps through the layers together.
//   kPath    : which of the launches this is (it returns at once unless the prepare kernel chose
//              it).  1: rows in LDS, updated in place: a layer is swept, barrier, written back to
//              the same row, barrier.  2: two rows in LDS alternate, one barrier per layer.
//              0: two rows of kHalo + pitch floats in `rows` in global memory, one candidate per
//              workgroup.  (A row that can be updated in place always fits the smaller LDS
//              allocation and two longer ones never do, so path 1 is exactly the in-place case
//              of a workgroup of the usual size; each instantiation holds only its own way of
//              stepping through a layer.)
//              3 (D record): path 1's code in a workgroup of twice the waves with up to a whole
//              compute unit's LDS: rows of up to twice path 1's length are still updated in
//              place (one candidate per workgroup, one workgroup per compute unit at a time).
//              4 (D record): path 0's code in a workgroup of twice the waves with a whole compute
//              unit's LDS for the window (its tiles are twice as long).
//   kNarrow  : S <= 64, one lane per level: the next layer's table is loaded without dependent
//              loads while a layer is swept (a separate instantiation, so that the waits of the
//              two ways of loading do not meet in one control-flow join)
//   kBlocks  : the checkpoint / block passes of the small-record solve (D record only); the
//              plain instantiation ignores `blocks`
//   kTodo    : behind dp_core, only the candidates it gave up (a separate instantiation: the test
//              for them changes how the compiler lays out and schedules the loops of the other
//              calls; B = 10^5, K = 128 was 1.5 % slower with it)
//   kTurns   : the workgroups that share a compute unit take turns at the instruction priority
//              (see the layer loop); `units` is the number of compute units
//   kSplit   : launched with twice the waves the plan was made for (D record, in place, S <= 64,
//              no more candidates than compute units, so a workgroup has its unit to itself and
//              one wave per SIMD and candidate issues too little).  Wave w of the second half is
//              the twin of wave w of the first: same team, same chunks, the other pairs of each
//              layer's entries (see fill_group_quads).  The second half only sweeps; tables,
//              record, row and the final argmin are the first half's.  The partial rows of the
//              second half lie in LDS behind the smaller allocation (the launch gets twice that).
// `pitch` is the record's row pitch (elements per (k, l) row).
struct FillShared {      // static LDS of the kernels
    float best[kMaxFillWaves];
    int time[kMaxFillWaves];
    // per team and for two layers: the entries (D record, at most one team per planned wave), or in the
    // same storage one 64-bit set of levels to visit (level record); a sweep looks kLookAhead entries too far
    __attribute__((aligned(8))) int2 entries[2 * kFillWaves * kWave + kLookAhead];
};
static_assert(sizeof(FillShared) <= kLdsStatic, "static LDS");
template <bool kLevel, int kPath, bool kNarrow, bool kBlocks, bool kTodo, bool kTurns, bool kSplit,
          bool kPairs, bool kBatched = false>
__device__ __forceinline__ void fill_candidates(
    ErrSource src, const int32_t *__restrict__ meta, LevelTables tables, int units, int K, int L,
    int S, int pitch, uint8_t *__restrict__ choice, float *__restrict__ drec,
    float *__restrict__ rows, int32_t *__restrict__ tstar, float *__restrict__ cost, Resume resume,
    Blocks blocks, Todo todo, float *lds, FillShared &sh)
{
    auto &s_best = sh.best;
    auto &s_time = sh.time;
    auto &s_entries = sh.entries;
    constexpr bool kGlobal = kPath == 0 || kPath == 4;     // rows in global memory
    constexpr bool kLds = !kGlobal, inplace = kPath == 1 || kPath == 3;
    static_assert(kPath < 3 || (!kLevel && !kBlocks && !kTurns && !kSplit),
                  "the launches of twice the waves are plain D-record fills");
    constexpr bool kQuads = !kLevel && kNarrow;  // the D-record sweep with 128-bit LDS reads
    constexpr bool kCanTile = !kLevel && !kBlocks && !kTodo && !(kPath == 1 && kNarrow);
    static_assert(!kSplit || (kQuads && kPath == 1 && !kBlocks && !kTurns),
                  "the split launch is the plain in-place D-record fill");
    if (meta[kMetaPath] != kPath || (kCanTile && meta[kMetaTiles] != 0))
        return;                                  // another launch does the work (or dp_tiles)
    const int bp = meta[kMetaBudget];
    const int tid = threadIdx.x, nthreads = blockDim.x;
    if (bp < 0) {                                // even the fastest levels exceed the budget
        if (tid == 0 && !(kBlocks && blocks.pass == 1) &&
            (!kTodo || todo.has_wave(blockIdx.x, K, L)))
            write_result<kTodo>(__builtin_inff(), 0, blockIdx.x, tstar, cost);
        return;
    }
    tables.limit = kGlobal ? bp : INT32_MAX;     // only the tiles of global rows depend on it
    const int teams = meta[kMetaTeams];
    const int tw = meta[kMetaTeamWaves];
    if ((long long)blockIdx.x * teams >= K)
        return;                                  // the first ceil(K / teams) workgroups suffice
    if constexpr (kTodo && kLevel) {             // (dp_rest has looked)
        bool any = false;
        for (int i = 0; i < teams && blockIdx.x * teams + i < (unsigned)K; ++i)
            any |= todo.has_wave(blockIdx.x * teams + i, K, L);
        if (!any)
            return;                              // solved already
    }
    const int row = meta[kMetaRow];
    const int lane = tid & (kWave - 1);
    int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    int half = 0;                                // kSplit: 1 for the twins of the planned waves
    if constexpr (kSplit) {
        const int planned = nthreads / (2 * kWave);
        half = wave >= planned ? 1 : 0;
        wave -= half * planned;
    }
    const bool lead = half == 0;
    const int team = wave / tw;
    const int wv = wave - team * tw;             // this wave's index in its team
    // Which share of the row this wave sweeps.  The low chunks of a row cost less than the high
    // ones (fewer levels reach them), and wave w of a workgroup runs on SIMD w mod 4: with the
    // shares in wave order one SIMD would hold the cheap shares of every team and another the
    // expensive ones.  Every second group of four waves therefore takes its shares in reverse.
    const bool mirrored = (tw & (tw - 1)) == 0 && ((wave >> 2) & 1);
    const int share = mirrored ? wv ^ (min(tw, 4) - 1) : wv;
    const int k = blockIdx.x * teams + team;
    const bool active = team < teams && k < K && (!kTodo || todo.has_wave(k, K, L));

    // rows: [apron | row] once (in place) or twice per team
    const int stride = kHalo + (kLds ? row : pitch);
    const int team_floats = inplace ? stride : (kLds ? 2 * stride : 0);    // (in LDS)
    float *base = kLds ? lds + (size_t)(team < teams ? team : 0) * team_floats
                       : rows + (size_t)blockIdx.x * 2 * stride;
    float *buf0 = base + kHalo;
    float *buf1 = inplace ? buf0 : buf0 + stride;

    // D before the first layer: time 0 costs nothing, nothing else is reachable (Eq. 3 then is
    // the general update).  -0.0f + e returns e bit for bit for every e, +0.0f would not for
    // e = -0.0f.  Aprons and chunks a layer does not compute keep this +inf.
    if constexpr (kLds) {
        for (int i = tid; i < teams * team_floats; i += nthreads)
            lds[i] = (i % team_floats == kHalo) ? -0.0f : __builtin_inff();
    } else {
        for (int i = tid; i < kHalo + row; i += nthreads) {
            base[i] = (i == kHalo) ? -0.0f : __builtin_inff();
            base[(size_t)stride + i] = __builtin_inff();
        }
    }
    __syncthreads();

    const int32_t *nact = meta + kMetaHeader + L;
    const size_t ke = active ? k : 0;            // candidate whose errors this wave reads

    // a candidate that shares its first l0 layers with the incumbent starts from the incumbent's
    // row l0 - 1, placed where layer l0 reads its previous row
    const int l0 = active ? resume.start(k, L) : 0;
    if (l0 > 0 && lead) {
        float *dst = (l0 & 1) ? buf1 : buf0;
        const float *from = resume.inc_rec + (size_t)(l0 - 1) * pitch;
        const int n = nact[l0 - 1] * kWave;
        for (int t = wv * kWave + lane; t < n; t += tw * kWave)
            dst[t] = from[t];
        if (wv == 0 && lane == 0 && dst != buf0)
            buf0[0] = __builtin_inff();          // undo the layer-0 start value
    }
    if (resume.first_layer)
        __syncthreads();
    // a block pass starts from the checkpoint below the block
    const int lb = kBlocks ? blocks.begin : 0;   // layers [lb, le) are filled
    const int le = kBlocks ? blocks.end : L;
    if constexpr (kBlocks) {
        if (lb > 0) {
            float *dst = (lb & 1) ? buf1 : buf0;
            const float *from =
                blocks.ckpt + (ke * blocks.slots + (size_t)(lb / blocks.stride - 1)) * pitch;
            const int n = nact[lb - 1] * kWave;
            if (active)
                for (int t = wv * kWave + lane; t < n; t += tw * kWave)
                    dst[t] = from[t];
            if (active && wv == 0 && lane == 0 && dst != buf0)
                buf0[0] = __builtin_inff();      // undo the layer-0 start value
            __syncthreads();
        }
    }

    // this candidate's part of the inputs and of the record
    const ErrSource mine = src.of_candidate(ke, L, S);
    uint8_t *choice_k = kLevel ? choice + ke * L * pitch : nullptr;
    float *drec_k = kLevel ? nullptr : drec + ke * L * pitch;
    if constexpr (kBlocks)
        drec_k = blocks.pass == 0 ? blocks.ckpt + ke * blocks.slots * pitch
                                  : blocks.block + ke * blocks.stride * pitch;

    // lane i keeps visited entry i of the layer being swept; the next layer's is fetched early
    const int s8 = tables.s8;
    // S <= 64: the first wave of a team prepares, for the next layer, the team's table of merged
    // errors (D record) or the set of levels worth visiting (level record)
    const bool producer = kNarrow && share == 0 && team < teams && lead;
    // kSplit: where the twins of this wave's team leave their minima
    float *part = kSplit ? lds + kLdsHalf / (int)sizeof(float) + (size_t)(team < teams ? team : 0) * row
                         : nullptr;
    unsigned long long *keep =
        reinterpret_cast<unsigned long long *>(&s_entries[0]) + (team < teams ? team : 0);
    int2 *const table = &s_entries[(team < teams && !kLevel ? team : 0) * kWave];
    constexpr int kNextTable = kFillWaves * kWave;   // from an even layer's table to an odd one's
    constexpr int kMax = group_limit<kLevel, kTurns>();
    // Rows in memory: chunks of a tile of layer l, whose window in LDS holds the layer's largest shift; fewer
    // than one per wave: there is no room for any, and the layer is swept from memory.
    auto tile_of = [&](int l) {
        const int span = meta[kMetaHeader + (2 + (size_t)kRangeStride) * L + l];
        const int tile = (meta[kMetaStage] / (int)sizeof(float) - span - 8) / kWave / tw * tw;
        return min(tile, tw * kMax);
    };
    auto unit = [&](int l) { return kGlobal && tile_of(l) < tw ? 1u : (unsigned)sizeof(float); };
    LevelEntry next_first{INT32_MAX, 0.0f};
    LevelFetch next_fetch{INT32_MAX, 0.0f, 0};
    if constexpr (kNarrow) {
        next_fetch = fetch_levels<kLevel>(tables.layer(lb), mine.layer(lb, S), S, s8, lane,
                                          producer);
        if (producer) {
            if constexpr (kLevel) {
                const unsigned long long visit =
                    levels_to_visit(next_fetch, load_twins(tables.layer(lb)), lane);
                if (lane == 0)
                    keep[(lb & 1) * kMaxFillWaves] = visit;
            } else {
                publish_entries(table + (lb & 1) * kNextTable, next_fetch, unit(lb), S, lane);
            }
        }
        __syncthreads();
    } else {
        next_first = load_level<kLevel>(tables.layer(lb), mine.layer(lb, S), s8, 0, lane);
    }
    Pending{&next_fetch, &next_first}.settle();   // no load is in flight at the loop's head
    // chunk boundaries of this wave
    const int32_t *range = meta + kMetaHeader + 2 * L + (size_t)lb * kRangeStride + share;
    int c_next = range[0], c_end_next = range[1];
    constexpr bool kWhole = kQuads && kPath == 1 && !kSplit;
    int whole_next = kWhole ? range[kWholeWord] : 0;
    // Two workgroups share a compute unit, and the hardware serves the older one first: left
    // alone, the first `units` workgroups of a launch run at full speed, the second `units` on what
    // is left and then by themselves, at barely more than half the unit's LDS rate.  The
    // instruction priority therefore alternates between the two halves of the last 2 * units
    // workgroups with the wall clock (100 MHz; 2^13 ticks = 82 us per turn), so both advance
    // alike and finish together.  Earlier workgroups of a longer launch are left alone: a
    // compute unit then always holds an older and a younger one, and a new one takes over when
    // the older is done.  A launch with no more workgroups than compute units has no pairs.
    // (kTurns: a separate instantiation, launched for batches of one or two rounds of
    // workgroups; the other one is exactly the code without any of this.)
    const unsigned turn = ((unsigned)blockIdx.x / (unsigned)units) & 1u;
    const int nwg = (K + teams - 1) / teams;
    const bool take_turns = kTurns && nwg > units && (long long)blockIdx.x + 2 * units >= nwg;
    unsigned long long now = take_turns ? wall_clock64() : 0;
    for (int l = lb; l < le; ++l) {
        if constexpr (kTurns) {
            if (take_turns) {
                if ((turn ^ (unsigned)(now >> kPriorityTurn)) & 1u)
                    __builtin_amdgcn_s_setprio(1);
                else
                    __builtin_amdgcn_s_setprio(0);
                now = wall_clock64();            // read now, looked at a layer later: no wait
            }
        }
        LevelEntry first = next_first;
        if constexpr (kNarrow) {
            first.shift = next_fetch.shift;
            if constexpr (kLevel) {
                first.err = next_fetch.raw;
                first.keep = keep[(l & 1) * kMaxFillWaves];
            }
        }
        if (l + 1 < le) {
            const LayerTable tn = tables.layer(l + 1);
            const ErrRow en = mine.layer(l + 1, S);
            // Rows in memory need all of their registers for the sweep: addresses of a lane that stayed in
            // registers over all layers (these, and with the level record those of the copy to LDS below) drove
            // four others to scratch memory.  (dp_rest keeps the index of a thread besides.)
            int mine_of = lane;
            if constexpr (kGlobal || (kTodo && !kLevel))
                asm("" : "+v"(mine_of));
            if constexpr (kNarrow)
                next_fetch = fetch_levels<kLevel>(tn, en, S, s8, mine_of, producer);
            else
                next_first = load_level<kLevel>(tn, en, s8, 0, mine_of);
        }
        const float *prev = (l & 1) ? buf1 : buf0;
        float *cur = (l & 1) ? buf0 : buf1;
        int c = 0, c_end = 0, whole = 0;         // this wave's chunks of the row
        if (active && l >= l0) {
            c = c_next;
            c_end = c_end_next;
            whole = whole_next;
        }
        if (l + 1 < le) {                        // the next layer's, read a layer ahead
            range += kRangeStride;
            c_next = range[0];
            c_end_next = range[1];
            if constexpr (kWhole)
                whole_next = range[kWholeWord];
        }
        uint8_t *choice_l = kLevel ? choice_k + (size_t)l * pitch : nullptr;
        float *drec_l = kLevel ? nullptr : drec_k + (size_t)l * pitch;
        if constexpr (kBlocks) {
            if (blocks.pass == 1)
                drec_l = drec_k + (size_t)(l - lb) * pitch;
            else if ((l + 1) % blocks.stride == 0 && l + 1 < L)
                drec_l = drec_k + (size_t)((l + 1) / blocks.stride - 1) * pitch;
            else
                drec_l = nullptr;                // this row is not kept
        } else if constexpr (!kLevel) {
            __builtin_assume(drec_l != nullptr);
        }
        const LayerTable tl = tables.layer(l);
        const ErrRow er = mine.layer(l, S);
        const int2 *const entries = table + (l & 1) * kNextTable;
        const Pending pending{&next_fetch, &next_first};
        if (kWhole && whole != 0) {
            fill_share_n<!kTodo, kBatched>(whole, cur, drec_l, first, entries, lane, pending);
        } else if constexpr (inplace) {          // c_end - c <= kMax by construction
            fill_group_n<kLevel, true, kMax, kQuads, kSplit, kPath == 1, false, kPairs, kBatched>(
                min(c_end - c, kMax), prev, cur, choice_l, drec_l, first, entries, tl, er, s8,
                c * kWave, lane, pending, half, part);
        } else {
            // Rows in global memory: the row is computed in tiles of at most kMax chunks per
            // wave, and the part of the previous row a tile reads (the tile itself and the
            // layer's largest usable shift to its left) is first copied to LDS, so the sweep
            // reads LDS as in the resident case.  One candidate per workgroup here, so every
            // wave takes the same number of trips.
            const int tile = kGlobal ? tile_of(l) : 0;
            const int span = kGlobal ? meta[kMetaHeader + (2 + (size_t)kRangeStride) * L + l] : 0;
            if (kGlobal && tile >= tw) {
                const int n_l = (active && l >= l0) ? nact[l] : 0;
                if (n_l == 0)
                    pending.settle();
                for (int c0 = 0; c0 < n_l; c0 += tile) {
                    const int nt = min(tile, n_l - c0);
                    // (lo a multiple of four floats: rows and aprons are, so the copy moves 16
                    // bytes per lane, eight loads in flight per lane; four floats more than the
                    // largest shift, for the lane left of a group's first quad)
                    const int lo = max(((c0 * kWave - span) & ~3) - 4, -kHalo);
                    const int len4 = ((c0 + nt) * kWave - lo) / 4;
                    const float4 *from = reinterpret_cast<const float4 *>(prev + lo);
                    float4 *to = reinterpret_cast<float4 *>(lds);
                    for (int i0 = 0; i0 < len4; i0 += 8 * nthreads) {
                        float4 v[8];
                        int first_quad = i0 + tid;
                        if constexpr (kLevel)     // (not eight of them in registers over all layers)
                            asm("" : "+v"(first_quad));
#pragma unroll
                        for (int j = 0; j < 8; ++j)   // (past the end: the last element again)
                            v[j] = from[min(first_quad + j * nthreads, len4 - 1)];
#pragma unroll
                        for (int j = 0; j < 8; ++j) {
                            const int i = first_quad + j * nthreads;
                            if (i < len4)
                                to[i] = v[j];
                        }
                    }
                    __syncthreads();
                    const int cb = c0 + (int)((long long)share * nt / tw);
                    const int ce = c0 + (int)((long long)(share + 1) * nt / tw);
                    fill_group_n<kLevel, false, kMax, kQuads, false, false, false, kPairs, kBatched>(
                        ce - cb, lds - lo, cur, choice_l, drec_l, first, entries, tl, er, s8,
                        cb * kWave, lane, pending);
                    __syncthreads();             // the next tile overwrites the staged part
                }
            } else {
                while (c < c_end) {
                    const int n = c_end - c;
                    const int groups = (n + kMax - 1) / kMax;
                    const int r = (n + groups - 1) / groups;
                    fill_group_n<kLevel, false, kMax, kQuads, false, false, kGlobal, kPairs, kBatched>(
                        r, prev, cur, choice_l, drec_l, first, entries, tl, er, s8, c * kWave, lane,
                        pending);
                    c += r;
                }
            }
        }
        // the table of the next layer; the barrier that ends this layer publishes it
        if (producer && l + 1 < le) {
            if constexpr (kLevel) {
                const unsigned long long visit =
                    levels_to_visit(next_fetch, load_twins(tables.layer(l + 1)), lane);
                if (lane == 0)
                    keep[((l + 1) & 1) * kMaxFillWaves] = visit;
            } else {
                publish_entries(table + ((l + 1) & 1) * kNextTable, next_fetch, unit(l + 1), S, lane);
            }
        }
        __syncthreads();
    }

    if constexpr (kBlocks) {
        if (blocks.pass == 1)
            return;                              // the final time is known from pass 0
    }
    // final argmin over t' <= bp within each team
    const float *last = (L & 1) ? buf1 : buf0;
    float bv = __builtin_inff();
    int bt = INT32_MAX;
    if (active && lead)
        for (int t = wv * kWave + lane; t <= bp; t += tw * kWave)
            argmin_merge(bv, bt, last[t], t);
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const float ov = __shfl_down(bv, off, kWave);
        const int ot = __shfl_down(bt, off, kWave);
        argmin_merge(bv, bt, ov, ot);
    }
    if (lane == 0 && lead) {
        s_best[wave] = bv;
        s_time[wave] = bt;
    }
    __syncthreads();
    if (active && lead && wv == 0 && lane == 0) {
        for (int w = 1; w < tw; ++w)
            argmin_merge(bv, bt, s_best[wave + w], s_time[wave + w]);
        write_result<kTodo>(bv, bt, k, tstar, cost);
    }
}

template <bool kLevel, int kPath, bool kNarrow, bool kBlocks, bool kTodo = false,
          bool kTurns = false, bool kSplit = false, bool kPairs = false>
__global__ __launch_bounds__(fill_waves<kLevel>() * (kSplit || kPath >= 3 ? 2 : 1) * kWave,
                             kLevel ? 8 : 4)
void dp_fill(
    ErrSource src, const int32_t *__restrict__ meta, LevelTables tables, int units, int K, int L,
    int S, int pitch, uint8_t *__restrict__ choice, float *__restrict__ drec,
    float *__restrict__ rows, int32_t *__restrict__ tstar, float *__restrict__ cost, Resume resume,
    Blocks blocks, Todo todo)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ FillShared sh;
    fill_candidates<kLevel, kPath, kNarrow, kBlocks, kTodo, kTurns, kSplit, kPairs>(
        src, meta, tables, units, K, L, S, pitch, choice, drec, rows, tstar, cost, resume, blocks,
        todo, lds, sh);
}

#include "dp_tiles.h"

// Final argmin for other budgets on an already filled D record: the rows hold exact-time costs
// and do not depend on the budget, so a smaller budget only shortens the range of the argmin
// (Sec. 3.2: the answer is min over t <= T of the last row).  One workgroup per candidate and
// budget; the time found (-1: none) is left in tstar[j * K + k] for the walk back.
struct Budgets {
    int32_t at[kCoreBudgets];
};
__global__ __launch_bounds__(256) void dp_budget_argmin(const int32_t *__restrict__ meta,
                                                        const float *__restrict__ drec, int K,
                                                        int L, int pitch, Budgets budgets,
                                                        int32_t *__restrict__ tstar, Todo todo)
{
    __shared__ float s_best[4];
    __shared__ int s_time[4];
    const int solve = blockIdx.x, j = solve / K, k = solve - j * K, tid = threadIdx.x;
    if (!todo.has_wave(solve, K, L))
        return;
    const int budget = budgets.at[j];
    const int bp = meta[kMetaBudget];
    // reduced budget: t' <= budget - M, and never beyond what the fill computed
    const long long reduced = (long long)budget - meta[kMetaMinTime];
    long long top = reduced < bp ? reduced : bp;
    if (bp >= 0) {
        const long long computed = (long long)meta[kMetaHeader + 2 * L - 1] * kWave - 1;
        top = top < computed ? top : computed;
    }
    float bv = __builtin_inff();
    int bt = INT32_MAX;
    if (bp >= 0) {
        const float *last = drec + ((size_t)k * L + (L - 1)) * pitch;
        for (int t = tid; t <= top; t += blockDim.x)
            argmin_merge(bv, bt, last[t], t);
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const float ov = __shfl_down(bv, off, kWave);
        const int ot = __shfl_down(bt, off, kWave);
        argmin_merge(bv, bt, ov, ot);
    }
    if ((tid & (kWave - 1)) == 0) {
        s_best[tid / kWave] = bv;
        s_time[tid / kWave] = bt;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < 4; ++w)
            argmin_merge(bv, bt, s_best[w], s_time[w]);
        tstar[solve] = bv < __builtin_inff() ? bt : -1;
    }
}

// The same for candidate k by one wave, which gets the time in every lane.
__device__ __forceinline__ int budget_time(const int32_t *__restrict__ meta, const float *__restrict__ drec, int k,
                                           int L, int pitch, int budget)
{
    const int lane = threadIdx.x & (kWave - 1), bp = meta[kMetaBudget];
    if (bp < 0)
        return -1;
    const long long reduced = (long long)budget - meta[kMetaMinTime];
    const long long computed = (long long)meta[kMetaHeader + 2 * L - 1] * kWave - 1;
    long long top = reduced < bp ? reduced : bp;
    top = top < computed ? top : computed;
    float bv = __builtin_inff();
    int bt = INT32_MAX;
    const float *const last = drec + ((size_t)k * L + (L - 1)) * pitch;
    constexpr int kLoads = 16;                   // at once
    const int end = (int)top;
    for (int t0 = lane; t0 <= end; t0 += kLoads * kWave) {
        float v[kLoads];
#pragma unroll
        for (int i = 0; i < kLoads; ++i)         // (past the end: the last one again)
            v[i] = last[min(t0 + i * kWave, end)];
#pragma unroll
        for (int i = 0; i < kLoads; ++i)
            argmin_merge(bv, bt, v[i], min(t0 + i * kWave, end));
    }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const float ov = __shfl_xor(bv, off, kWave);
        const int ot = __shfl_xor(bt, off, kWave);
        argmin_merge(bv, bt, ov, ot);
    }
    return __builtin_amdgcn_readfirstlane(bv < __builtin_inff() ? bt : -1);
}

// ---------------------------------------------------------------------------------------------
// Walk back (last loop of Alg. 1).  kByItself: not enqueued by the call that filled the record, whose
// workspace may therefore have been scratch since; it then holds no table, and t* anything.  (Not a
// run-time flag: the load that it guards was issued all the same, 0.3 us of a walk of 6 us.)

// Level record: one wave per candidate, two layers a trip to memory.  With the level of layer l at time t all levels
// of layer l - 1 that it may lead to are read, lane s the one at t - shift_s, and what these lead on by is there
// before.  us a walk, a lane per candidate, which reads a level, then its shift, then the next level, and so: L = 54,
// S = 40, B = 10^4, K = 1 29.7 and 16.7, K = 1024 68.5 and 27.0, K = 4096 91.9 and 50.6; L = 400, S = 2, K = 4000 478
// and 299; L = 30, S = 100, K = 600 37.5 and 18.0.  The cost is re-summed over the profile in layer order (exactly
// the sum Alg. 1's strict "<" sweep carries to the cell).
// kLevelBlocks: see LayerLevels.
template <int kLevelBlocks> struct LevelShifts {
    int shift[kLevelBlocks];
    __device__ __forceinline__ void load(const int32_t *__restrict__ tau, const int32_t *__restrict__ meta, int l,
                                         int S, int lane)
    {
        const int m = meta[kMetaHeader + l];
#pragma unroll
        for (int b = 0; b < kLevelBlocks; ++b)
            shift[b] = tau[(size_t)l * S + min(b * kWave + lane, S - 1)] - m;
    }
};
// Level s of what the lanes hold.
template <int kLevelBlocks> __device__ __forceinline__ int of_level(const int (&held)[kLevelBlocks], int s)
{
    int v = from_lane(held[0], s & (kWave - 1));
#pragma unroll
    for (int b = 1; b < kLevelBlocks; ++b)
        if (s / kWave == b)
            v = from_lane(held[b], s & (kWave - 1));
    return v;
}

template <int kLevelBlocks, bool kByItself>
__global__ __launch_bounds__(kWalkThreads) void dp_backtrace_levels(
    const int32_t *__restrict__ tau, ErrSource src, const int32_t *__restrict__ meta,
    const uint8_t *__restrict__ choice, const int32_t *__restrict__ tstar, int K, int L, int S, int pitch,
    int16_t *__restrict__ profile, float *__restrict__ cost, Todo todo)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int k = uniform((int)(blockIdx.x * (kWalkThreads / kWave) + threadIdx.x / kWave));
    if (k >= K || !todo.has_wave(k, K, L))
        return;
    int16_t *prof = profile + (size_t)k * L;
    int t = uniform(tstar[k]);
    const bool none = kByItself && !meta[kMetaTable];
    if (none || t < 0) {
        for (int l = lane; l < L; l += kWave)
            prof[l] = none ? -2 : -1;
        if (none && lane == 0)
            cost[k] = __builtin_nanf("");
        return;
    }
    const uint8_t *choice_k = choice + (size_t)k * L * pitch;
    LevelShifts<kLevelBlocks> upper, lower;
    upper.load(tau, meta, L - 1, S, lane);
    lower.load(tau, meta, max(L - 2, 0), S, lane);
    bool ok = true;
    for (int l = L - 1; l >= 0; l -= 2) {
        int level[kLevelBlocks];
        const int here = choice_k[(size_t)l * pitch + t];
#pragma unroll
        for (int b = 0; b < kLevelBlocks; ++b) {
            level[b] = kNoLevel;
            // (a time that the lane's level leads to, or none)
            if (l > 0 && b * kWave + lane < S && upper.shift[b] <= t)
                level[b] = choice_k[(size_t)(l - 1) * pitch + (t - upper.shift[b])];
        }
        const LevelShifts<kLevelBlocks> upper_now = upper, lower_now = lower;
        upper.load(tau, meta, max(l - 2, 0), S, lane);
        lower.load(tau, meta, max(l - 3, 0), S, lane);
        // a level that there is not, or that leads below time 0: cannot happen on a filled table
        const int s = uniform(here);
        ok = s < S;
        if (!ok)
            break;
        t -= of_level(upper_now.shift, s);
        ok = t >= 0;
        if (lane == 0)
            prof[l] = (int16_t)s;
        if (!ok || l == 0)
            break;
        const int below = of_level(level, s);
        ok = below < S;
        if (!ok)
            break;
        t -= of_level(lower_now.shift, below);
        ok = t >= 0;
        if (!ok)
            break;
        if (lane == 0)
            prof[l - 1] = (int16_t)below;
    }
    const float sum = ok ? profile_cost(src.of_candidate(k, L, S), L, S, prof) : __builtin_nanf("");
    if (lane == 0)
        cost[k] = sum;
}

// The same by one lane per candidate, which reads a level, then its shift, then the next level: what a trip takes
// counts less the more waves there are, and these are 64 times fewer.
template <bool kByItself>
__global__ void dp_backtrace_levels_by_lanes(const int32_t *__restrict__ tau, ErrSource src,
                                             const int32_t *__restrict__ meta,
                                             const uint8_t *__restrict__ choice,
                                             const int32_t *__restrict__ tstar, int K, int L, int S,
                                             int pitch, int16_t *__restrict__ profile,
                                             float *__restrict__ cost, Todo todo)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= K || !todo.has(k, K, L))
        return;
    int16_t *prof = profile + (size_t)k * L;
    int t = tstar[k];
    const bool none = kByItself && !meta[kMetaTable];
    if (none || t < 0) {
        for (int l = 0; l < L; ++l)
            prof[l] = none ? -2 : -1;
        if (none)
            cost[k] = __builtin_nanf("");
        return;
    }
    const int32_t *mn = meta + kMetaHeader;
    const uint8_t *choice_k = choice + (size_t)k * L * pitch;
    bool ok = true;
    for (int l = L - 1; ok && l >= 0; --l) {
        const int s = choice_k[(size_t)l * pitch + t];
        prof[l] = (int16_t)s;
        ok = s < S;          // cannot fail on a filled table; never index tau out of range
        if (ok) {
            t -= tau[(size_t)l * S + s] - mn[l];
            ok = t >= 0;
        }
    }
    __threadfence_block();
    float acc = ok ? -0.0f : __builtin_nanf("");
    for (int l = 0; ok && l < L; ++l)
        acc += src.row(k, l, L, S).at(prof[l]);
    cost[k] = acc;
}
// Up to how many candidates a unit has a wave for each.  us a walk by lanes and by waves, L = 54, S = 40: K = 8192 67
// and 44, 12000 71 and 61, 16384 82 and 85, 32768 131 and 179; L = 24, S = 130: K = 8192 30 and 28, 12000 31 and 38;
// L = 8, S = 20: K = 4096 7.7 and 7.4, 6000 7.8 and 8.4, 16384 11 and 17; L = 4, S = 4, K = 200000 15 and 98.
constexpr int kLevelWaves = 32, kLevelWavesShort = 16, kLevelShort = 16;

// One wave walks solve `solve`, which is candidate k under some budget, from the time that tstar() gives.
template <int kLevelBlocks, bool kByItself, bool kGuess = false, class Time>
__device__ __forceinline__ void walk_table(const int32_t *__restrict__ tau, ErrSource src,
                                           const int32_t *__restrict__ meta,
                                           const float *__restrict__ drec, Time tstar,
                                           int solve, int k, int L, int S, int pitch,
                                           int16_t *__restrict__ profile, float *cost,
                                           Resume resume)
{
    const int lane = threadIdx.x & (kWave - 1);
    int16_t *prof = profile + (size_t)solve * L;
    const ErrSource mine = src.of_candidate(k, L, S);
    const float *drec_k = drec + (size_t)k * L * pitch;
    const int l0 = resume.start(k, L);           // rows below l0 are the incumbent's
    auto row_of = [&](int l) { return (l < l0 ? resume.inc_rec : drec_k) + (size_t)l * pitch; };
    const int from = kByItself && !meta[kMetaTable] ? -2 : tstar();
    int t;
    if constexpr (kGuess)
        t = walk_guessed(tau, mine, meta, row_of, from, L, S, prof);
    else
        t = walk_layers<kLevelBlocks>(tau, mine, meta, row_of, from, 0, L, L, S, prof);
    if (t < 0) {
        if (lane == 0)
            cost[solve] = t == -1 ? __builtin_inff() : __builtin_nanf("");
        return;
    }
    const float acc = profile_cost(mine, L, S, prof);
    if (lane == 0)
        cost[solve] = acc;
}

// `budgets` > 1 (solve_budgets): solve j * K + k is candidate k under budget j, and its final time
// comes in through cost (dp_budget_argmin).
// kGuess: see walk_guessed.
template <int kLevelBlocks, bool kByItself, bool kGuess>
__global__ __launch_bounds__(kWalkThreads) void dp_backtrace_values(
    const int32_t *__restrict__ tau, ErrSource src, const int32_t *__restrict__ meta,
    const float *__restrict__ drec, const int32_t *tstar, int K, int budgets, int L, int S,
    int pitch, int16_t *__restrict__ profile, float *cost, Resume resume, Todo todo)
{
    int solve = blockIdx.x * (kWalkThreads / kWave) + threadIdx.x / kWave;
    if constexpr (kGuess)
        solve = uniform(solve);
    const int k = budgets > 1 ? solve % K : solve;
    if (solve < K * budgets && todo.has_wave(solve, K, L))
        walk_table<kLevelBlocks, kByItself, kGuess>(
            tau, src, meta, drec, [=]() __attribute__((always_inline)) { return tstar[solve]; }, solve, k, L, S,
            pitch, profile, cost, resume);
}

// ---------------------------------------------------------------------------------------
// The walk of a candidate that has a compute unit to itself: one workgroup.  A wave that gathers its
// levels' entries of the row below waits for memory once per layer, 0.63 us, because where it reads next
// follows from what it read.  Which part of the rows below it can come to is known ahead, though: i layers
// below time t, [t - the largest shifts of those layers, t] (a layer's smallest shift is 0).  So a block of up to
// kLoneBlock layers is taken at a time, as many as have all their windows in LDS: every wave copies its
// share of them (memory to LDS, 256 floats an instruction, all in flight at once), then wave 0 walks
// through LDS, about 0.12 us a layer, while the other waves fetch the levels of the next block.  Windows
// grow by one layer's shifts from row to row; with few to a block a copy costs what it saves, and the
// rows are read entry by entry as before (kLoneLeast).
// us a walk, launch included, one wave by itself and so: K = 1, L = 54, S = 40, B = 10^4 (12 layers a block)
// 33.2 and 21.0, B = 10^5 (windows too wide, entry by entry) 41.5 and 36.6; L = 17, S = 200, B = 10^4 22.6 and
// 14.4; L = 400, S = 2 215 and 101; L = 10, S = 8, B = 1000 11.8 and 11.5.  About 0.15 us a layer is a copy's
// share of the time, the rest instructions of wave 0 one after the other: a step that read a window's place and
// bounds from several tables, with branches around what is out of bounds, took 0.28 us (28.6 us a walk).
// ---------------------------------------------------------------------------------------
constexpr int kLoneWaves = 16;
constexpr int kLoneBlock = kLoneWaves - 1;      // layers of a block: waves 1 to 15 fetch one's levels each
constexpr int kLoneLeast = 4;                   // fewest layers that are copied for
constexpr int kPiece = 4 * kWave;               // floats of one copy
// A window's sum counts no more than this of a shift, so that 15 of them fit; a window whose sum has come to it
// begins at bucket 0.
constexpr int kFarShift = 1 << 27;
template <int kLevelBlocks> constexpr int kLonePieces = kLevelBlocks == 1 ? 140 : 92;

template <int kLevelBlocks>
struct LoneShared {
    __attribute__((aligned(16))) float window[kLonePieces<kLevelBlocks> * kPiece + 4];   // and row -1's -0
    // What wave 0 needs at layer top - i for a level, in one read.  Where windows are copied: x, what to take
    // from its place in the window above (from the time, for i = 0) for the place in this one; y, the error;
    // z, the floats of the window; w, where it begins.  Otherwise x is the shift and z the row's end.  z = 0
    // past S.  (Row kLoneBlock: read ahead and not used.)
    int4 step[kLoneBlock + 1][kLevelBlocks * kWave];
    int highest[kLoneBlock], reach[kLoneBlock];          // largest shift of layer top - i, row below it
    int t;
    float target;
};
static_assert(sizeof(LoneShared<1>) <= 160 * 1024 && sizeof(LoneShared<4>) <= 160 * 1024, "LDS");
static_assert((long long)kLoneBlock * kFarShift <= INT32_MAX, "sums of a window");

template <int kLevelBlocks, bool kByItself>
__global__ __launch_bounds__(kLoneWaves * kWave) void dp_backtrace_alone(
    const int32_t *__restrict__ tau, ErrSource src, const int32_t *__restrict__ meta,
    const float *__restrict__ drec, const int32_t *tstar, int K, int budgets, int L, int S,
    int pitch, int16_t *__restrict__ profile, float *cost, Resume resume)
{
    constexpr int kMost = kLonePieces<kLevelBlocks>;
    __shared__ LoneShared<kLevelBlocks> sh;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int solve = blockIdx.x, k = budgets > 1 ? solve % K : solve;
    int16_t *prof = profile + (size_t)solve * L;
    const ErrSource mine = src.of_candidate(k, L, S);
    const float *drec_k = drec + (size_t)k * L * pitch;
    const int l0 = resume.start(k, L);           // rows below l0 are the incumbent's
    auto row_of = [&](int l) { return (l < l0 ? resume.inc_rec : drec_k) + (size_t)l * pitch; };

    // wave 1 + i holds the levels of layer top - i
    LayerLevels<kLevelBlocks> levels{};
    auto fetch = [&](int top) {
        const int i = wave - 1;
        if (i < 0 || i > top)
            return;
        levels = load_layer<kLevelBlocks>(tau, mine.layer(top - i, S), meta, top - i, L, S, lane);
        int high = 0;
#pragma unroll
        for (int b = 0; b < kLevelBlocks; ++b)   // (INT32_MAX past S)
            high = max(high, b * kWave + lane < S ? levels.shift[b] : 0);
        high = wave_scan(high, 0, Larger{});
        if (lane == kWave - 1) {
            sh.highest[i] = min(high, kFarShift);
            sh.reach[i] = levels.reach;
        }
    };

    int t = kByItself && !meta[kMetaTable] ? -2 : tstar[solve];
    t = __builtin_amdgcn_readfirstlane(t);
    float target = t >= 0 ? row_of(L - 1)[t] : 0.0f;
    fetch(L - 1);
    if (threadIdx.x == 0)
        sh.window[kMost * kPiece] = -0.0f;
    __syncthreads();             // tstar may be the words of the costs: every wave has read its own
    if (t < 0) {
        for (int l = threadIdx.x; l < L; l += kLoneWaves * kWave)
            prof[l] = t == -1 ? -1 : -2;         // -1: no profile meets the budget
        if (threadIdx.x == 0)
            cost[solve] = t == -1 ? __builtin_inff() : __builtin_nanf("");
        return;
    }

    for (int top = L - 1; top >= 0;) {
        // lane i plans the window of the row below layer top - i, in pieces
        const bool here = lane < kLoneBlock && lane <= top, rows = here && lane < top;
        const int i = min(lane, kLoneBlock - 1);
        const int reach = here ? sh.reach[i] : 0;
        const int high = wave_scan(here ? sh.highest[i] : 0, 0, Add{});
        const int from = rows && high < min(t, kFarShift) ? (t - high) & ~3 : 0;
        const int last = min(t, reach - 1);
        const int pieces = rows && last >= from ? min((last - from) / kPiece, kMost) + 1 : 0;
        const int ends = wave_scan(pieces, 0, Add{});
        const int held = __popcll(__ballot(here && ends <= kMost));
        const bool copied = held >= min(kLoneLeast, top + 1);
        const int n = copied ? held : min(kLoneBlock, top + 1);
        const int begin = rows ? (ends - pieces) * kPiece : kMost * kPiece;
        const int width = rows ? max(min(pieces * kPiece, reach - from), 0) : min(reach, 1);
        if (copied) {
            // the first of the row's floats that are copied; and their end, a whole number of fours
            const float *start = row_of(rows ? top - 1 - lane : 0) + from;
            const int start_lo = (int)reinterpret_cast<uintptr_t>(start);
            const int start_hi = (int)(reinterpret_cast<uintptr_t>(start) >> 32);
            const int all = __builtin_amdgcn_readlane(ends, n - 1);
            for (int p = wave; p < all; p += kLoneWaves) {
                const int r = __popcll(__ballot(lane < n && ends <= p));     // the row of piece p
                const int u = p * kPiece - __builtin_amdgcn_readlane(begin, r) + 4 * lane;
                const uintptr_t at = (uintptr_t)(unsigned)__builtin_amdgcn_readlane(start_hi, r) << 32 |
                                     (unsigned)__builtin_amdgcn_readlane(start_lo, r);
                if (u < __builtin_amdgcn_readlane(width, r))
                    __builtin_amdgcn_global_load_lds(
                        (const __attribute__((address_space(1))) void *)(
                            reinterpret_cast<const float *>(at) + u),
                        (__attribute__((address_space(3))) void *)(sh.window + p * kPiece), 16, 0, 0);
            }
        }
        if (wave > 0) {
            const int r = wave - 1, above = r > 0 ? __builtin_amdgcn_readlane(from, max(r - 1, 0)) : 0;
            const int by = copied ? __builtin_amdgcn_readlane(from, r) - above : 0;
            const int z = __builtin_amdgcn_readlane(copied ? width : reach, r);
            const int w = __builtin_amdgcn_readlane(begin, r);
#pragma unroll
            for (int b = 0; b < kLevelBlocks; ++b)
                sh.step[r][b * kWave + lane] =
                    int4{(int)((unsigned)levels.shift[b] + by), __float_as_int(levels.err[b]),
                         b * kWave + lane < S ? z : 0, w};
        }
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        if (wave > 0) {
            fetch(top - n);
        } else {
            int at = t, found_of = -1;           // lane r: the level of layer top - r
            bool damaged = false;
            auto steps = [&](auto entry) __attribute__((always_inline)) {
                int4 next[kLevelBlocks];
#pragma unroll
                for (int b = 0; b < kLevelBlocks; ++b)
                    next[b] = sh.step[0][b * kWave + lane];
                for (int r = 0; r < n; ++r) {
                    unsigned u[kLevelBlocks];
                    float pv[kLevelBlocks], err[kLevelBlocks];
                    bool valid[kLevelBlocks];
#pragma unroll
                    for (int b = 0; b < kLevelBlocks; ++b) {
                        u[b] = (unsigned)at - (unsigned)next[b].x;
                        valid[b] = u[b] < (unsigned)next[b].z;
                        pv[b] = entry(r, u[b], valid[b], next[b]);
                        err[b] = __int_as_float(next[b].y);
                    }
#pragma unroll
                    for (int b = 0; b < kLevelBlocks; ++b)
                        next[b] = sh.step[r + 1][b * kWave + lane];
                    int found = -1, to = 0;
                    float value = 0.0f;
#pragma unroll
                    for (int b = kLevelBlocks - 1; b >= 0; --b) {
                        const unsigned long long mask = __ballot(valid[b] && pv[b] + err[b] == target);
                        if (mask) {              // (the lowest level there is)
                            const int first = __builtin_ctzll(mask);
                            found = b * kWave + first;
                            to = __builtin_amdgcn_readlane((int)u[b], first);
                            value = lane_value(pv[b], first);
                        }
                    }
                    damaged = found < 0;         // (cannot happen on a filled record)
                    if (damaged)
                        return;
                    found_of = lane == r ? found : found_of;
                    at = to;
                    target = value;
                }
            };
            if (copied)
                steps([&](int, unsigned u, bool, int4 s) __attribute__((always_inline)) {
                    return sh.window[(unsigned)s.w + min(u, (unsigned)s.z)];
                });
            else
                steps([&](int r, unsigned u, bool valid, int4) __attribute__((always_inline)) {
                    const float *row = row_of(max(top - r - 1, 0));
                    return top == r ? -0.0f
                           : valid ? __builtin_nontemporal_load(&row[u]) : __builtin_inff();
                });
            if (lane < n)
                prof[top - lane] = (int16_t)found_of;
            if (lane == 0) {
                sh.t = damaged ? -2 : at + (copied ? __builtin_amdgcn_readlane(from, n - 1) : 0);
                sh.target = target;
            }
        }
        __syncthreads();
        t = __builtin_amdgcn_readfirstlane(sh.t);
        target = sh.target;
        if (t == -2) {
            for (int l = lane; wave == 0 && l < L; l += kWave)
                prof[l] = -2;
            if (threadIdx.x == 0)
                cost[solve] = __builtin_nanf("");
            return;
        }
        top -= n;
    }
    if (wave > 0)
        return;
    const float acc = profile_cost(mine, L, S, prof);
    if (lane == 0)
        cost[solve] = acc;
}

// The walk through one block of layers [blocks.begin, blocks.end) of the small-record solve: rows
// come from the block record, the row below the block from its checkpoint; tstar holds the time
// to start from and receives the time below the block; the cost is summed after the first block
// (the last one walked).
template <int kLevelBlocks>
__device__ __forceinline__ void walk_block(const int32_t *__restrict__ tau, ErrSource src,
                                           const int32_t *__restrict__ meta,
                                           int32_t *__restrict__ tstar, int k, int L, int S,
                                           int pitch, int16_t *__restrict__ profile,
                                           float *__restrict__ cost, Blocks blocks)
{
    const int lane = threadIdx.x & (kWave - 1);
    int16_t *prof = profile + (size_t)k * L;
    const ErrSource mine = src.of_candidate(k, L, S);
    const int lb = blocks.begin;
    const float *const rows = blocks.block + (size_t)k * blocks.stride * pitch;
    const float *const below =
        lb > 0 ? blocks.ckpt + ((size_t)k * blocks.slots + (lb / blocks.stride - 1)) * pitch : rows;
    auto row_of = [=](int l) { return l >= lb ? rows + (size_t)(l - lb) * pitch : below; };
    const int t = walk_layers<kLevelBlocks>(tau, mine, meta, row_of, tstar[k], lb, blocks.end, L, S,
                                            prof);
    if (lane == 0) {
        tstar[k] = t;                            // -2: the blocks below are marked the same way
        if (t == -2)
            cost[k] = __builtin_nanf("");
    }
    if (t < 0 || lb > 0)
        return;
    const float acc = profile_cost(mine, L, S, prof);
    if (lane == 0)
        cost[k] = acc;
}

template <int kLevelBlocks>
__global__ __launch_bounds__(kWalkThreads) void dp_backtrace_blocks(
    const int32_t *__restrict__ tau, ErrSource src, const int32_t *__restrict__ meta,
    int32_t *__restrict__ tstar, int K, int L, int S, int pitch, int16_t *__restrict__ profile,
    float *__restrict__ cost, Blocks blocks)
{
    const int k = blockIdx.x * (kWalkThreads / kWave) + threadIdx.x / kWave;
    if (k < K)
        walk_block<kLevelBlocks>(tau, src, meta, tstar, k, L, S, pitch, profile, cost, blocks);
}

// Behind dp_core, D record: fill and walk back of the few candidates it gave up, under one or several budgets or
// with checkpoints, in one launch, or two or three where rows may be longer than a workgroup of the usual size has in
// place.  Nearly always there is nothing to do, and what counts is the number of launches, 1.9 us each and more with
// many workgroups.  us a call with a launch for each step and row length, and so:
// Nothing given up, L = 54, S = 40, B = 10^4: with checkpoints K = 64 56 and 45, K = 300 77 and 49, K = 1024 106 and
// 72, K = 256, L = 200, S = 64, B = 65536 219 and 194; 64 candidates under six budgets 56.6 and 53.4; under one, K = 1024
// 74 and 72.  Eleven of 1024 given up: 384 and 379, with checkpoints 720 and 700.  All of them: K = 64 364 and 364, K = 700
// 726 and 780, K = 1024 941 and 943; with checkpoints K = 300 981 and 918, K = 1024 1812 and 1851, L = 200 29600 and
// 27900, K = 300, B = 60000 3860 and 3730, B = 15000 1190 and 1260; 64 candidates under six budgets 386 and 399.  (K = 700
// and B = 15000 are the worst of 80 shapes.)
//   kShape 0: no more candidates than compute units, one to a workgroup; rows of any length.  A candidate has a unit
//             to itself then whatever LDS its workgroup asks for, and its walk only needs its own rows.
//          1: more of them, rows in place (path 1), two workgroups to a unit, `teams` candidates to each
//          2: more of them, longer rows; with checkpoints those that fit LDS (path 2)
//          3: with checkpoints, rows in memory (path 0), whose workgroups take half of a unit's LDS each
// The arguments are read again where a fill or a walk begins.  Kept from block to block, they and what is made of them
// took all scalar registers, the rest of which moved to lanes of vector registers and back within the sweep:
// eleven of 1024 given up took 433 us, all of K = 250, L = 30, S = 100, B = 9000 with checkpoints 1410 (969 so).
struct Rest {
    ErrSource src;
    LevelTables tables;
    int units, K, L, S, pitch;
    float *drec, *rows;
    int32_t *tstar;
    int16_t *profile;
    float *cost;
    Resume resume;
    Blocks blocks;
    Todo todo;
    int budgets;                 // 0: one, and its walk; several, and theirs; -1: the walks are other launches'
    Budgets budget;
};
template <bool kNarrow, bool kBlocks, int kShape>
__global__ __launch_bounds__((kBlocks || kShape == 1 ? 1 : 2) * kFillWaves * kWave, 4) void dp_rest(
    const int32_t *__restrict__ tau, const int32_t *__restrict__ meta, const Rest)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ FillShared sh;
    constexpr int kLevelBlocks = kNarrow ? 1 : 4;
    constexpr int kRestAt = 2 * sizeof(void *);  // behind tau and meta
    auto args = []() __attribute__((always_inline)) {
        auto at = __builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(at));             // (an address of its own: read anew)
        return *(const Rest *)((const char *)at + kRestAt);
    };
    auto budget_of = [](int j) __attribute__((always_inline)) {
        return *(const int32_t *)((const char *)__builtin_amdgcn_kernarg_segment_ptr() + kRestAt +
                                  offsetof(Rest, budget) + j * sizeof(int32_t));
    };
    auto teams_of = [=]() __attribute__((always_inline)) { return kShape == 1 ? meta[kMetaTeams] : 1; };
    {
        const Rest a = args();
        const int path = meta[kMetaPath];
        if ((kShape > 0 && (path == 1) != (kShape == 1)) ||
            (kBlocks && kShape > 1 && (path == 2) != (kShape == 2)))
            return;
        const int teams = teams_of(), first = blockIdx.x * teams;
        bool any = false;
        for (int i = 0; i < teams && first + i < a.K; ++i)
            any |= a.todo.has_wave(first + i, a.K, a.L);
        if (!any)
            return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    int pass = 0, begin = 0, end = 0;             // with checkpoints: pass 1 for each block of layers [begin, end)
    auto fill = [&](auto path) __attribute__((always_inline)) {
        constexpr int kPath = decltype(path)::value;
        Rest a = args();
        if constexpr (kBlocks) {
            a.blocks.pass = pass;
            a.blocks.begin = begin;
            a.blocks.end = pass == 0 ? a.L : end;
        }
        fill_candidates<false, kPath, kNarrow, kBlocks, true, kShape == 1,
                        kPath == 1 && kNarrow && !kBlocks && kShape == 0, false, kBlocks && (kShape == 1 || kShape == 2)>(
            a.src, meta, a.tables, a.units, a.K, a.L, a.S, a.pitch, nullptr, a.drec, a.rows, a.tstar,
            a.budgets ? nullptr : a.cost, a.resume, a.blocks, a.todo, lds, sh);
    };
    for (;;) {
        if constexpr (kShape < 2)                 // (each only where the path is its own)
            fill(Many<1>{});
        if constexpr (kShape == 0 || kShape == 2)
            fill(Many<kBlocks ? 2 : 3>{});
        if constexpr (kShape == 0 || kShape == (kBlocks ? 3 : 2))
            fill(Many<kBlocks ? 0 : 4>{});
        __syncthreads();                          // the rows and the final time are written
        if constexpr (!kBlocks)
            break;
        Rest a = args();
        if (pass == 1) {
            const int teams = teams_of(), k = blockIdx.x * teams + wave;
            a.blocks.begin = begin;
            a.blocks.end = end;
            if (wave < teams && k < a.K && a.todo.has_wave(k, a.K, a.L))
                walk_block<kLevelBlocks>(tau, a.src, meta, a.tstar, k, a.L, a.S, a.pitch, a.profile, a.cost,
                                         a.blocks);
            __syncthreads();                      // the block's rows are read
            if (begin == 0)
                return;
            end = begin;
        } else {
            pass = 1;
            end = a.L;
        }
        begin = (end - 1) / a.blocks.stride * a.blocks.stride;
    }
    const Rest a = args();
    const int teams = teams_of(), first = blockIdx.x * teams, waves = blockDim.x / kWave;
    for (int i = wave; a.budgets >= 0 && i < teams * max(a.budgets, 1); i += waves) {
        const int j = i / teams, k = first + (i - j * teams), solve = j * a.K + k;
        if (k >= a.K || __builtin_amdgcn_readfirstlane(a.profile[(size_t)solve * a.L]) != kGivenUp)
            continue;
        const int t = a.budgets ? budget_time(meta, a.drec, k, a.L, a.pitch, budget_of(j)) : a.tstar[k];
        walk_table<kLevelBlocks, false>(
            tau, a.src, meta, a.drec, [=]() __attribute__((always_inline)) { return t; }, solve, k, a.L, a.S, a.pitch,
            a.profile, a.cost, a.resume);
    }
}

int launch_status()
{
    return hipGetLastError() == hipSuccess ? SPDY_DP_OK : SPDY_DP_ERR_LAUNCH;
}

// What the host keeps per device between calls: the number of compute units (asked once, not per
// solve) and where this device's copy of `scratch` lives.
constexpr int kMaxDevices = 64;
struct DeviceState {
    int units = 0;
    void *scratch = nullptr;
};
std::mutex g_device_lock;
DeviceState g_device[kMaxDevices];

// The current device's state; `with_scratch` also resolves the device address of `scratch`.
// Returns SPDY_DP_OK or SPDY_DP_ERR_LAUNCH (the runtime refused a query).
int device_state(bool with_scratch, DeviceState *out)
{
    int device = 0;
    if (hipGetDevice(&device) != hipSuccess || device < 0 || device >= kMaxDevices)
        return SPDY_DP_ERR_LAUNCH;
    std::lock_guard<std::mutex> hold(g_device_lock);
    DeviceState &st = g_device[device];
    if (st.units <= 0) {
        int units = 0;
        if (hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, device) !=
                hipSuccess || units <= 0)
            return SPDY_DP_ERR_LAUNCH;
        st.units = units;
    }
    if (with_scratch && !st.scratch) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr)
            return SPDY_DP_ERR_LAUNCH;
        st.scratch = ptr;
    }
    *out = st;
    return SPDY_DP_OK;
}

// A call whose workspace is scratch: its candidates go through dp_core first.
struct CoreCall {
    int16_t *profile;                 // [budgets][K][L]
    float *cost;                      // [budgets][K]
    const int32_t *budget;            // host, [budgets]
    int budgets;
    unsigned char *spill;             // the record's memory
    size_t spill_bytes;
    bool rest;                        // dp_rest does what is left
    bool walks;                       // also the walks under several budgets
};

// LDS and limits of dp_core for these sizes; false where the full table has to be used at once.
// The staged tables, L * S pairs, have to fit LDS.  What a row may span is taken from the LDS that a
// workgroup can have without lowering how many a compute unit holds (registers allow four).  On
// the timing tables of the performance cases' kinds (2729 candidates, L = 8 - 48, counted on the
// host) the widest row of one candidate in a hundred spans 3 B / L buckets and more, of none
// 4.8 B / L, so no more than 6 B / L is asked for.  Where there is less than 4 B / L, rows that need more lie in memory, which an
// instantiation of its own allows for (4 % slower where none does: the registers).  Giving such a
// candidate up costs most of the reduced solve and then the whole table: L = 17, S = 14, B = 43125, K = 20:
// 235 us with eight of them given up, 132 with the rows in LDS, 124 for the full table at
// once; L = 11, S = 9, B = 30006, K = 1407 (806 given up): 329, 211 with rows in memory, 272.
// Rows are not worth any price, though: fewer than one candidate in a thousand needed a sixteenth of the
// sweeps of the full table, and a table that needs more (ties everywhere, errors linear in the
// times) is given up there, after as long again as the full table takes at the worst measured.
constexpr int kCoreRecord = 8192;     // least LDS for the recorded entries
constexpr int kCoreWork = 4096;       // sweeps of 64 buckets in any case; one wave takes 20 ns for each
constexpr int kCorePerUnit = 4;       // workgroups that a compute unit has registers for
constexpr int kCoreStatic = 4096;     // static LDS of dp_core, rounded up
static_assert(sizeof(CoreShared) + 3 * 256 * sizeof(int32_t) + 128 <= kCoreStatic, "static LDS");
bool core_params(int L, int S, int B, long long workgroups, int units, CoreParams *cp, int *lds)
{
    if (L > kCoreMaxLayers || B > kCoreMaxBudget || S > 255)
        return false;
    int parts = 1;
    while (2 * parts * L <= kCoreThreads && 2 * parts <= kWave && parts < S)
        parts *= 2;
    cp->parts = parts;
    cp->parts_log2 = __builtin_ctz(parts);
    cp->share_log2 = 0;
    while ((2 << cp->share_log2) * L <= kWave && 2 << cp->share_log2 <= parts)
        ++cp->share_log2;
    cp->per_part = ((S + parts - 1) / parts + 3) / 4 * 4;
    cp->pad = parts * cp->per_part - S;
    if (cp->per_part > 128)
        return false;
    cp->step_layers = kCoreThreads / S;
    cp->pitch = (S + cp->pad) | 1;
    // (some 30 levels beyond one per layer are usual, nine per layer the most seen)
    const int room = 4 * L > 256 ? 4 * L : 256;
    cp->entries = L * S < room ? (L * S + 1) / 2 * 2 : room;
    const size_t lists = cp->entries * sizeof(CoreEntry) + (size_t)(L + 1) * sizeof(double) +
                         (size_t)L * (sizeof(CoreStep) + sizeof(float) + sizeof(int));
    const size_t staged = align_up((size_t)L * cp->pitch * sizeof(float2), 16);

    const long long rounds = (workgroups + units - 1) / units;
    // (LDS is given out in steps of 1280 bytes: a third of it, to the byte, fits only twice)
    const size_t share = rounds <= 1 ? (size_t)kLdsBytes
                                     : 160 * 1024 / (rounds < kCorePerUnit ? rounds : kCorePerUnit) /
                                               1280 * 1280 - kCoreStatic;
    const long long most = align_up((size_t)B + 1, kWave);
    long long wanted = (6LL * B / L > 1024 ? 6LL * B / L : 1024) / kWave * kWave;
    wanted = wanted < most ? wanted : most;
    const size_t row = sizeof(float) * kWave;     // (LDS is divided in these units)
    size_t table = (kCoreRecord + 2 * row * (wanted / kWave)) * 5 / 4;
    if (table + lists > share)
        table = share > lists ? share - lists : 0;
    const size_t least = kCoreRecord + 2 * row * ((most < 1024 ? most : 1024) / kWave);
    table = table > least ? table : least;
    table = (table > staged ? table : staged) / 16 * 16;
    if (table + lists > (size_t)kLdsBytes)
        return false;
    const size_t record = table / 5 > (size_t)kCoreRecord ? table / 5 : (size_t)kCoreRecord;
    const long long fit = (long long)((table - record) / (2 * row)) * kWave;
    cp->window = (int)(fit < most ? fit : most);
    cp->far = cp->window < most && cp->window < 4LL * B / L ? 1 : 0;        // (how far is for the caller, who knows the memory)
    cp->table_bytes = (int)table;
    cp->record = (int)(table - 2 * sizeof(float) * (size_t)cp->window);
    const long long part = (long long)L * S * (B / kWave + 1) / 16;
    cp->work = part < kCoreWork ? kCoreWork : (part < INT32_MAX / 2 ? (int)part : INT32_MAX / 2);
    size_t all = table + lists;
    // as many entries again where that does not change how many workgroups share a compute unit (deep networks
    // have candidates with five a layer)
    const size_t more = all + room * sizeof(CoreEntry);
    auto per_unit = [](size_t bytes) { return 160 * 1024 / align_up(bytes + kCoreStatic, 1280); };
    if (cp->entries == room && more <= (size_t)kLdsBytes && per_unit(more) == per_unit(all)) {
        cp->entries += room;
        all = more;
    }
    *lds = (int)all;
    return true;
}

// Where the full table is taken at once: tables of a handful of layers with short rows are through it
// before dp_core is through its dozen passes.
//   - Whatever the call, up to 256 candidates, in 0.1 us of latency: the table 1.2 us a layer for its barriers,
//     0.7 us for its hop of the walk back, 5000 updates in 0.1 us; dp_core 14 us and 0.6 us a layer (as both
//     were when the line was drawn).  us with the table and with dp_core, now: K = 1, L = 4, S = 10, B = 4351
//     22 and 25; K = 3, L = 5, S = 54, B = 382 24 and 24; K = 200, L = 8, S = 20, B = 1000 24 and 28; four
//     budgets, K = 61, L = 8, S = 51, B = 420 30 and 34; beyond the line K = 1, L = 8, S = 30, B = 1500 26 and
//     24, S = 40, B = 2000 31 and 23, K = 200, L = 12, S = 8, B = 500 24 and 25.
//   - Where one fill and one walk back are all that the table takes, more candidates, too: the slowest of them
//     sets dp_core's time, the table's hardly grows.  Of 631 drawn calls (L = 4 - 200) 58 were more than 5 %
//     slower than the better side without this line, 36 are with it.  Now K = 2247, L = 8, S = 10, B = 982 41
//     and 76; K = 428, L = 6, S = 16, B = 134 24 and 28; K = 1000, L = 9, S = 12, B = 2000 38 and 44; and on
//     the other side of where the line would lie today, K = 188, L = 9, S = 15, B = 15627 52 and 48, K = 300,
//     L = 9, S = 30, B = 1000 38 and 31, K = 2000, L = 10, S = 12, B = 1000 42 and 65 (not taken).  (Not for a
//     call that resumes from an incumbent: it may only be direct where the incumbent's call, K = 1, was
//     whatever entry point that went through, or there are no rows to take and every candidate is filled from
//     layer 0.  The first line is one of the sizes alone and holds for K = 1 where it holds for K.)
bool table_is_short(int K, int L, int S, int B, bool one_fill)
{
    const long long updates = (long long)L * S * (B + 1LL);
    if (K <= 256 && 19LL * L + updates / 5000 < 140 + 6LL * L)
        return true;
    return one_fill && K >= 8 && L <= 9 && L * S <= 300 && updates * ((K + 255LL) / 256) <= 4000000;
}

// Whether dp_small takes the call: a candidate's tables, rows and levels fit LDS, every candidate has a
// compute unit, and the whole takes less than 16 us by what was measured, 6 us and for every level of every
// layer 0.06 us, 0.08 more per 1000 buckets from 512 on.  Anything else takes 20 us and more.  K = 1 and 200,
// us a call with and without: L = S = 8, B = 256: 9.4 and 20.3, 9.7 and 24.2; L = S = 8, B = 1000: 12.7 and 21.1;
// beyond the line L = 8, S = 16, B = 1000: 18.9 and 22.5; L = S = 16, B = 256: 22.0 and 24.1; L = 8, S = 40,
// B = 1000: 36.7 and 26.2.
bool small_call(int K, int L, int S, int B)
{
    DeviceState dev;
    const long long beyond = B > 512 ? B - 512 : 0;
    return S <= kWave && L <= 256 && B < 1 << 16 && (long long)L * S * (60000 + 80 * beyond) <= 10000000 &&
           small_lds(L, S, B) <= (size_t)kSmallLds && device_state(false, &dev) == SPDY_DP_OK &&
           K <= dev.units;
}

int launch_small(const int32_t *tau, ErrSource src, int K, int L, int S, int B, int16_t *profile,
                 float *cost, int32_t *has_table, hipStream_t q)
{
    (void)hipGetLastError();
    const int threads = small_row(B) < 256 ? 256 : (small_row(B) < kSmallThreads ? small_row(B) : kSmallThreads);
    hipLaunchKernelGGL(dp_small, dim3(K), dim3(threads), small_lds(L, S, B), q, tau, src, L, S, B,
                       profile, cost, has_table);
    return launch_status();
}

// Whether dp_rest walks back under J budgets too: where each of its waves has one walk at most.  A walk waits for memory
// once a layer, and a second one behind it as long again.  us a call of eight candidates, all given up, L = 54, S = 40,
// B = 10^4, by launches of their own and so: six budgets 380 and 394 (and 57 and 53 where nothing is given up, K = 64),
// 64 budgets 407 and 690; K = 700, L = 30, S = 20, B = 1000, 16 budgets 229 and 290.
bool rest_walks(const Layout &lay, int K, int J, int units)
{
    const long long teams = (K + 2LL * units - 1) / (2LL * units);         // at most, of a workgroup
    const size_t waves = lay.row / kWave < (size_t)kFillWaves ? lay.row / kWave : (size_t)kFillWaves;
    return J * teams <= (long long)waves;
}

// Sets up the call for the J budgets, the largest of which `lay` is for; false: the full table at
// once.  `one_fill`: all that the full table would take is one fill and one walk back.
bool core_call(const Layout &lay, int K, int L, int S, const int32_t *budget, int J, bool one_fill,
               int16_t *profile, float *cost, void *workspace, size_t workspace_bytes,
               CoreCall *call)
{
    CoreParams cp{};
    int lds = 0, largest = 0;
    DeviceState dev;
    if (lay.status != SPDY_DP_OK || !workspace || device_state(false, &dev) != SPDY_DP_OK)
        return false;
    for (int j = 0; j < J; ++j)
        largest = budget[j] > largest ? budget[j] : largest;
    if (!core_params(L, S, largest, 1, 1, &cp, &lds) ||
        table_is_short(K, L, S, largest, one_fill))
        return false;
    *call = CoreCall{profile, cost, budget, J,
                     static_cast<unsigned char *>(workspace) + lay.record_off,
                     workspace_bytes - lay.record_off,
                     lay.variant == kValueRecord, rest_walks(lay, K, J, dev.units)};
    return true;
}

// Budgets that one launch takes with a workgroup of 256 threads per (candidate, budget): a grid of
// 2^32 threads is refused.
int budgets_per_launch(int K, int L)
{
    static_assert(kCoreThreads == 256, "2^24 workgroups are 2^32 threads");
    const long long fit = ((1LL << 24) - 1 - (L + 1LL)) / K;
    return fit < 1 ? 1 : (fit < kCoreBudgets ? (int)fit : kCoreBudgets);
}

int launch_core(const int32_t *tau, ErrSource src, int K, int L, int S, const PrepareArgs &prep,
                const CoreCall &call, int units, hipStream_t q)
{
    const int most = budgets_per_launch(K, L);
    for (int j0 = 0; j0 < call.budgets; j0 += most) {
        const int n = call.budgets - j0 < most ? call.budgets - j0 : most;
        const long long blocks = L + 1LL + (long long)K * n;
        CoreParams cp{};
        int lds = 0;
        if (!core_params(L, S, prep.B, blocks, units, &cp, &lds))
            return SPDY_DP_ERR_LAUNCH;           // callers ask first
        cp.budgets = n;
        for (int j = 0; j < n; ++j)
            cp.budget[j] = call.budget[j0 + j];
        const size_t each = call.spill_bytes / ((size_t)K * n) / 16 * 16;
        const bool far = cp.far != 0;
        if (far)                                 // half of the memory for two rows
            cp.far = (int)(each / 16 < prep.B + 1u ? each / 16 : prep.B + 1u);
        const size_t left = each - (far ? 2 * cp.far * sizeof(float) : 0);
        cp.spill = call.spill;
        constexpr size_t kMost = INT32_MAX / 16 * 16;        // (rows stay aligned)
        cp.spill_bytes = (long long)(left < kMost ? left : kMost);
        auto core = far ? dp_core<true> : dp_core<false>;
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(core),
                                hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) !=
            hipSuccess)
            return SPDY_DP_ERR_LAUNCH;
        hipLaunchKernelGGL(core, dim3((unsigned)blocks), dim3(kCoreThreads), lds, q, tau, src, K, L,
                           S, prep, cp, call.profile + (size_t)j0 * K * L,
                           call.cost + (size_t)j0 * K);
    }
    return launch_status();
}

template <bool kLevel, bool kNarrow, bool kBlocks, bool kPairs, bool kTodo>
int enqueue_fill(const Layout &lay, const int32_t *tau, ErrSource src, Resume resume, int K, int L,
                int S, int B, char *ws, float *cost, hipStream_t q, Blocks blocks,
                const CoreCall *core)
{
    int32_t *meta = reinterpret_cast<int32_t *>(ws + lay.meta_off);
    int32_t *shifts = reinterpret_cast<int32_t *>(ws + lay.shifts_off);
    int32_t *order = reinterpret_cast<int32_t *>(ws + lay.order_off);
    int32_t *start = reinterpret_cast<int32_t *>(ws + lay.start_off);
    int32_t *entry = reinterpret_cast<int32_t *>(ws + lay.entry_off);
    int32_t *tstar = reinterpret_cast<int32_t *>(ws + lay.tstar_off);
    uint8_t *choice = kLevel ? reinterpret_cast<uint8_t *>(ws + lay.record_off) : nullptr;
    float *drec = kLevel ? nullptr : reinterpret_cast<float *>(ws + lay.record_off);
    float *rows = reinterpret_cast<float *>(ws + (kLevel ? lay.rows_level : lay.rows_value));
    const int pitch = (int)lay.row;
    const int nchunks = pitch / kWave;
    const int s8 = (int)lay.s8;

    // The reduced row length is only known on the device, so the fill kernel is enqueued with an
    // LDS allocation that lets two workgroups share a compute unit and, if a row of the full
    // budget could need more, once more with a larger one (and once with the rows in global
    // memory if even that may not do); the prepare kernel picks the launch that fits and the
    // others return at once.  A row that the waves of a workgroup can hold in registers is
    // updated in place whatever the reduced length turns out to be, so one row bounds the need;
    // otherwise two rows alternate.
    // workgroups the chip holds at once: two per compute unit for either variant
    DeviceState dev;
    if (device_state(false, &dev) != SPDY_DP_OK)
        return SPDY_DP_ERR_LAUNCH;
    const int units = dev.units;
    // Workgroups that take turns at the priority pay off when a launch is one or two rounds of
    // workgroups (measured: K = 4 x units 4 % faster, 16 x units no gain and a slightly slower
    // kernel), and need pairs of workgroups to begin with.
    const bool turns = K > units && (long long)K <= 4LL * units;
    const int waves = nchunks < fill_waves<kLevel>() ? nchunks : fill_waves<kLevel>();
    const int max_group = turns ? group_limit<kLevel, true>() : group_limit<kLevel, false>();
    const size_t row_bytes = (lay.row + kHalo) * sizeof(float);
    const bool beyond_place = (long long)nchunks > (long long)waves * max_group;
    const size_t need = beyond_place ? 2 * row_bytes : row_bytes;
    const int lds_small = kLdsHalf;
    // D record: a row too long for the in-place launch may still be updated in place by a
    // workgroup of twice the waves that takes up to a whole compute unit's LDS (every length the
    // two-row launch could take is covered by it, so that launch is not enqueued then).
    constexpr bool can_widen = !kLevel && !kBlocks;
    const bool wide = can_widen && beyond_place;
    const int wide_waves = wide ? 2 * fill_waves<kLevel>() : 0;
    const int wide_group = group_limit<kLevel, false>();
    const int lds_wide = wide ? (int)(row_bytes < (size_t)kLdsBytes ? row_bytes : kLdsBytes) : 0;
    const int lds_large = (need <= (size_t)kLdsHalf || wide) ? 0
                          : (need <= (size_t)kLdsBytes ? (int)need : kLdsBytes);
    // whether the full budget's row may have to live in global memory (implies lay.may_spill)
    const bool in_memory =
        wide ? ((long long)nchunks > (long long)wide_waves * wide_group ||
                row_bytes > (size_t)kLdsBytes)
             : need > (size_t)kLdsBytes;
    auto in_place = turns ? dp_fill<kLevel, 1, kNarrow, kBlocks, kTodo && kLevel, true, false, kPairs>
                          : dp_fill<kLevel, 1, kNarrow, kBlocks, kTodo && kLevel, false, false, kPairs>;
    // Two workgroups to a unit, whose rows are folded for wide reads (dp_columns).  The level record only with
    // something to sweep, and not many candidates of few levels and layers, of which a unit has room for fewer: us a
    // solve by dp_fill and so, S = 12, L = 82, B = 920, K = 2655 386 and 452; S = 38, L = 11, B = 423, K = 4029 136
    // and 142; S = 70, L = 86, B = 304, K = 331 505 and 566; S = 25, L = 10, B = 2516, K = 3284 163 and 202; S = 17,
    // L = 14, B = 3357, K = 1144 126 and 137; and where it is taken S = 16, L = 124, B = 1585, K = 1534 691 and 646;
    // S = 35, L = 37, B = 833, K = 1378 246 and 191; S = 20, L = 9, B = 1396, K = 312 55 and 43; S = 33, L = 19,
    // B = 3271, K = 1890 269 and 244.
    // The budget's length counts, and not that of the reduced row: a workgroup of dp_fill has a wave for every chunk of the
    // budget, and where those are sixteen it is slower on short rows too.  us a fill by dp_fill and so, B = 3000, rows of
    // 250 buckets: S = 70, L = 86, K = 300 569 and 476, S = 16, L = 54, K = 1024 173 and 137, S = 40, L = 54, K = 4000
    // 388 and 347.  Slower on rows of one chunk with 65 to 100 levels (S = 70, K = 4000, L = 54 420 and 476) and for some
    // numbers of candidates beyond 4 x units on rows of 13 to 45 chunks, few levels above all (L = 20, K = 2100, 26
    // chunks: S = 16 175 and 206, S = 40 297 and 320).  Both launches, for the prepare kernel to choose from, would save
    // 0.2 % over 441 fills of more than 4 x units candidates, less than the idle one takes (2 us and more).
    // D record of more than 64 levels: always.  us by dp_fill and so, K = 4000: S = 65, L = 10, B = 800 179 and 150;
    // S = 255, L = 10, B = 800 390 and 306; S = 100, L = 12, B = 61 505 and 150; the worst of 370 on 1 - 80 chunks 0.92.
    constexpr bool kLeft = kTodo && kLevel, kRest = kTodo && !kLevel;      // (the D record's are dp_rest's)
    constexpr bool can_fold = (!kNarrow || (kLevel && kPairs)) && !kBlocks && !kTodo;
    const bool columns = can_fold && K > units && !resume.first_layer &&
                         (!kLevel || (S >= kFoldLevels && B >= kFoldBudget &&
                                      (K <= 4 * (long long)units || L * S >= kFoldWork)));
    // A candidate that has a compute unit to itself gets twice the waves (the second half takes
    // every other pair of each layer's entries and needs a second row in LDS for its minima).
    constexpr bool can_split = !kLevel && kNarrow && !kBlocks;       // (behind dp_core: dp_rest)
    const bool split = can_split && K <= units;
    int place_threads = waves * kWave, place_lds = lds_small;
    if (split) {
        place_threads *= 2;
        place_lds *= 2;
        static_assert(2 * kLdsHalf <= kLdsBytes, "two half allocations fit one workgroup");
    }
    if constexpr (can_split && !kTodo) {
        if (split) {
            in_place = dp_fill<kLevel, 1, kNarrow, kBlocks, kLeft, false, true>;
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(in_place),
                                    hipFuncAttributeMaxDynamicSharedMemorySize,
                                    kLdsBytes) != hipSuccess)
                return SPDY_DP_ERR_LAUNCH;
        }
    }
    auto two_rows = dp_fill<kLevel, 2, kNarrow, kBlocks, kLeft, false, false, kPairs>;
    auto wide_place = dp_fill<kLevel, can_widen ? 3 : 1, kNarrow, kBlocks, kLeft, false, false,
                              kPairs>;           // (3 when it exists)
    // The D record's global-row launch also has twice the waves (one workgroup per compute unit
    // with all of its LDS for the window; measured against two workgroups of the usual size with
    // half the LDS each: 11 % faster on a batch of four candidates per unit).
    const bool wide_global = can_widen && waves == fill_waves<kLevel>();
    const int global_waves = wide_global ? 2 * waves : waves;
    // (rows that may lie in memory are long: `waves` is the full number then)
    constexpr bool can_tile = !kLevel && !kBlocks && !kTodo;
    auto in_global = dp_fill<kLevel, can_widen ? 4 : 0, kNarrow, kBlocks, kLeft, false, false, kPairs>;
    if (!kRest && wide &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(wide_place),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) != hipSuccess)
        return SPDY_DP_ERR_LAUNCH;
    // always the same limit, so that calls from several host threads cannot undo each other's
    if (!kRest && lds_large &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(two_rows),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) != hipSuccess)
        return SPDY_DP_ERR_LAUNCH;
    // The global-row launch stages its tiles' windows in LDS: all of it with one workgroup per
    // compute unit; workgroups of the usual size take half of it when there are candidates for
    // two per unit (one sweeps while the other copies).
    const int lds_stage = (K > units && !wide_global) ? kLdsHalf : kLdsBytes;
    if (!kRest && in_memory &&
        hipFuncSetAttribute(reinterpret_cast<const void *>(in_global),
                            hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) != hipSuccess)
        return SPDY_DP_ERR_LAUNCH;

    // Several workgroups per candidate, or one with less to do between the layers (see dp_tiles.h): where each
    // has two compute units, and up to one per unit where rows are short (K = 256, L = 54, us so and by a
    // workgroup with all of its waves on one candidate: S = 40, B = 1000 71 and 123, B = 4000 132 and 164,
    // B = 8000 199 and 208, B = 10000 240 and 235, B = 16000 294 and 300; S = 20, B = 8000 159 and 173,
    // B = 10000 189 and 191, B = 16000 223 and 234); and where rows may have to lie in memory otherwise.
    const bool tiles_do = can_tile && !resume.first_layer &&
                          (2LL * K <= units || (K <= units && B <= kTileLone));
    const bool tiles_sure = tiles_do && B <= (kNarrow ? kTileSure : kTileSureWide);
    TileArgs ta{units, tiles_do ? 0 : 1, 0, (in_memory ? kLdsBytes : kTileLds) / (int)sizeof(float),
                nullptr, 0};
    if (tiles_do || (can_tile && !resume.first_layer && in_memory)) {
        ta.most = in_memory ? (K <= 512 ? kTileMost : (K <= 2048 ? 8192 / K : 4)) : units / K;
        ta.most = ta.most < kTileMost ? ta.most : kTileMost;
        // the books lie where the rows in memory would, or in tables that nothing else reads then; they
        // are for more than one tile only
        size_t room = 0;
        if (lay.may_spill) {
            ta.books = reinterpret_cast<int *>(rows);
            room = lay.total_value - lay.rows_value;
        } else if (kNarrow || tiles_sure) {
            ta.books = order;
            room = lay.entry_off - lay.order_off;
        }
        ta.room = (int)(room / sizeof(int) < (1u << 30) ? room / sizeof(int) : (1u << 30));
    }
    const PrepareArgs prep{2 * units, s8, B, waves, max_group, lds_small, lds_large, lds_stage,
                           kLevel ? 0 : (kNarrow ? 2 : (tiles_sure ? 3 : 1)), split ? 1 : 0, wide_waves, wide_group,
                           lds_wide, global_waves, kBlocks || core || resume.first_layer ? 0 : 1,
                           kTodo ? 0 : 1, !columns ? kNoColumns : (kLevel ? kLevelColumns : kValueColumns),
                           meta, shifts, order, start, entry, ta};
    Todo todo;
    if (core) {
        todo = Todo{core->profile, core->budgets};
        const int st = launch_core(tau, src, K, L, S, prep, *core, units, q);
        if (st != SPDY_DP_OK)
            return st;
    } else if (!(kBlocks && blocks.pass == 1)) { // the block passes reuse pass 0's tables
        hipLaunchKernelGGL(dp_prepare, dim3(L + 1), dim3(256), 0, q, tau, K, L, S, prep);
    }
    const LevelTables tables{shifts, order, start, entry, s8};
    if constexpr (kRest) {
        Rest rest{src, tables, units, K, L, S, pitch, drec, rows, tstar, core->profile, core->cost, resume, blocks,
                  todo, cost ? 0 : (core->walks ? core->budgets : -1), {}};
        for (int j = 0; j < rest.budgets; ++j)
            rest.budget.at[j] = core->budget[j];
        auto launch = [&](auto kernel, int threads, int lds) {
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) == hipSuccess)
                hipLaunchKernelGGL(kernel, dim3(K), dim3(threads), lds, q, tau, meta, rest);
        };
        const int threads = wide ? wide_waves * kWave : waves * kWave;
        int lds = lds_wide > lds_large ? lds_wide : lds_large;
        lds = in_memory && lds_stage > lds ? lds_stage : lds;
        if (K <= units) {
            launch(dp_rest<kNarrow, kBlocks, 0>, wide ? threads : place_threads, place_lds > lds ? place_lds : lds);
        } else {
            launch(dp_rest<kNarrow, kBlocks, 1>, waves * kWave, kLdsHalf);
            if constexpr (kBlocks) {              // (rows may be longer)
                if (lds_large)
                    launch(dp_rest<kNarrow, kBlocks, 2>, threads, lds_large);
                if (in_memory)
                    launch(dp_rest<kNarrow, kBlocks, 3>, threads, lds_stage);
            } else if (lds > 0) {
                launch(dp_rest<kNarrow, kBlocks, 2>, threads, lds);
            }
        }
        return launch_status();
    }
    if constexpr (can_tile) {
        if (ta.most > 0 && !in_memory) {
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(dp_tiles),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kTileLds) !=
                hipSuccess)
                return SPDY_DP_ERR_LAUNCH;
            const long long most = (long long)K * ta.most;
            hipLaunchKernelGGL(dp_tiles, dim3((unsigned)(most < units ? most : units)),
                               dim3(kTileThreads), kTileLds, q, src, meta, tables, K, L, S, pitch,
                               drec, tstar, cost, ta.books);
        }
    }
    if (tiles_sure)
        return launch_status();
    if constexpr (can_fold) {
        if (columns) {
            auto folded = turns ? dp_columns<kLevel, true, kNarrow ? 1 : 4>
                                : dp_columns<kLevel, false, kNarrow ? 1 : 4>;
            hipLaunchKernelGGL(folded, dim3(K), dim3(kFillWaves * kWave), kLdsHalf, q, src, meta, tables, units,
                               K, L, S, pitch, choice, drec, tstar, cost);
        }
    }
    if (!columns && (!kNarrow || !tiles_do))
        hipLaunchKernelGGL(in_place, dim3(K), dim3(place_threads), place_lds, q, src, meta, tables,
                           units, K, L, S, pitch, choice, drec, rows, tstar, cost, resume, blocks,
                           todo);
    if (wide && !(can_tile && in_memory))
        hipLaunchKernelGGL(wide_place, dim3(K), dim3(wide_waves * kWave), lds_wide, q, src, meta,
                           tables, units, K, L, S, pitch, choice, drec, rows, tstar, cost, resume,
                           blocks, todo);
    if constexpr (can_tile) {
        if (in_memory) {
            auto wide_or_tiles = dp_wide<kNarrow>;
            if (hipFuncSetAttribute(reinterpret_cast<const void *>(wide_or_tiles),
                                    hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes) !=
                hipSuccess)
                return SPDY_DP_ERR_LAUNCH;
            hipLaunchKernelGGL(wide_or_tiles, dim3(ta.most > 0 && K < units ? units : K),
                               dim3(kTileThreads), kLdsBytes, q, src, meta, tables, units, K, L, S,
                               pitch, drec, tstar, cost, resume, ta.books);
        }
    }
    if (lds_large)
        hipLaunchKernelGGL(two_rows, dim3(K), dim3(waves * kWave), lds_large, q, src, meta, tables,
                           units, K, L, S, pitch, choice, drec, rows, tstar, cost, resume, blocks, todo);
    if (in_memory)
        hipLaunchKernelGGL(in_global, dim3(K), dim3(global_waves * kWave), lds_stage, q, src, meta, tables,
                           units, K, L, S, pitch, choice, drec, rows, tstar, cost, resume, blocks, todo);
    return launch_status();
}

template <bool kLevel, bool kNarrow, bool kBlocks = false, bool kPairs = false>
int launch_fill(const Layout &lay, const int32_t *tau, ErrSource src, Resume resume, int K, int L,
                int S, int B, char *ws, float *cost, hipStream_t q, Blocks blocks,
                const CoreCall *core)
{
    auto launch = core ? enqueue_fill<kLevel, kNarrow, kBlocks, kPairs, true>
                       : enqueue_fill<kLevel, kNarrow, kBlocks, kPairs, false>;
    return launch(lay, tau, src, resume, K, L, S, B, ws, cost, q, blocks, core);
}

int validate(const Layout &lay, const void *workspace)
{
    if (lay.status != SPDY_DP_OK)
        return lay.status;
    if (!workspace)
        return SPDY_DP_ERR_NULL;
    return SPDY_DP_OK;
}

int fill_impl(const int32_t *tau, ErrSource src, int K, int L, int S, int B, float *cost,
              void *workspace, size_t workspace_bytes, void *stream, Resume resume = Resume{},
              const CoreCall *core = nullptr)
{
    if (!tau || (!cost && !core))
        return SPDY_DP_ERR_NULL;
    const Layout lay = make_layout(K, L, S, B, workspace_bytes);
    const int st = validate(lay, workspace);
    if (st != SPDY_DP_OK)
        return st;
    hipStream_t q = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace);
    (void)hipGetLastError();
    auto launch = S <= kWave ? launch_fill<false, true> : launch_fill<false, false>;
    if (lay.variant == kLevelRecord)
        launch = S > kWave        ? launch_fill<true, false, false, true>
                 : S >= kPairsFrom ? launch_fill<true, true, false, true>
                                   : launch_fill<true, true, false, false>;
    return launch(lay, tau, src, resume, K, L, S, B, ws, cost, q, Blocks{}, core);
}

void launch_walk(const int32_t *tau, ErrSource src, const int32_t *meta, const float *drec,
                 const int32_t *tstar, int K, int budgets, int L, int S, int pitch,
                 int16_t *profile, float *cost, Resume resume, Todo todo, bool by_itself,
                 int units, hipStream_t q)
{
    // A unit to every candidate, whose LDS the windows take: us a walk by a wave's guesses and so, L = 54, S = 40,
    // B = 10^4: K = 1 26.0 and 23.0, K = 64 31.3 and 24.7, K = 256 34.2 and 33.9; L = 200, S = 64, B = 3000, K = 250
    // 92.7 and 62.9 (a wave layer by layer: K = 1 33.2, K = 256 47.4); beyond, workgroups would queue for units.
    // (Behind dp_core hardly any candidate is left to walk.  Copies are of 16 bytes: a record that does not lie
    // so is walked entry by entry.)
    // The price: it waits for a unit whose LDS is free, where four waves without LDS would start beside a fill
    // of another stream.  us a step, the walk of one step beside the fill of the next, four waves layer by layer
    // and so: K = 64 165 and 137, K = 100 155 and 166, K = 192 211 and 225, K = 256 258 and 234; K = 200, L = 30,
    // S = 100, B = 12000 326 and 473.  On one stream: 169 and 142, 194 and 168, 251 and 231, 253 and 236, 352
    // and 345.
    auto whole = [](const void *p) { return reinterpret_cast<uintptr_t>(p) % 16 == 0; };
    if (!todo.profile && K * (long long)budgets <= units && whole(drec) && whole(resume.inc_rec)) {
        auto alone = S <= kWave ? dp_backtrace_alone<1, false> : dp_backtrace_alone<4, false>;
        if (by_itself)
            alone = S <= kWave ? dp_backtrace_alone<1, true> : dp_backtrace_alone<4, true>;
        hipLaunchKernelGGL(alone, dim3(K * budgets), dim3(kLoneWaves * kWave), 0, q, tau, src, meta,
                           drec, tstar, K, budgets, L, S, pitch, profile, cost, resume);
        return;
    }
    const int per_block = kWalkThreads / kWave;
    auto walk = S <= kWave ? dp_backtrace_values<1, false, false> : dp_backtrace_values<4, false, false>;
    if (by_itself)
        walk = S <= kWave ? dp_backtrace_values<1, true, false> : dp_backtrace_values<4, true, false>;
    // By guesses from kGuessLayers on and up to kGuessWaves candidates to a unit, beyond which the waves that a unit
    // holds at once have two each.  us a walk, layer by layer and so, of tables at falling returns and of tables where
    // most guesses fail (errors like the root of the time saved): K = 1024, S = 40 L = 24 24 and 20, 24 and 30; L = 32
    // 31 and 23, 31 and 33; L = 48 44 and 30, 44 and 45; L = 54 50 and 33, 50 and 55; K = 600, S = 8, L = 40 36 and 30,
    // 36 and 42; L = 48 43 and 34, 42 and 46; L = 80 68 and 45, 67 and 66.  S = 40: K = 4096, L = 54 76 and 50, L = 24
    // 32 and 28; K = 6000 75 and 73, 35 and 42; K = 16384, L = 30 98 and 110.  (Going on layer by layer after a few
    // wrong guesses was not kept: with both walks in it the kernel took 55 where this takes 35.)
    // Rows of 2 GB and more, whose buckets a buffer does not reach, and the few candidates that the reduced solve
    // leaves: layer by layer.
    if (S <= kWave && L >= kGuessLayers && pitch < 1 << 29 && !todo.profile &&
        (long long)K * budgets <= (long long)kGuessWaves * units)
        walk = by_itself ? dp_backtrace_values<1, true, true> : dp_backtrace_values<1, false, true>;
    hipLaunchKernelGGL(walk, dim3((K * budgets + per_block - 1) / per_block), dim3(kWalkThreads), 0,
                       q, tau, src, meta, drec, tstar, K, budgets, L, S, pitch, profile, cost,
                       resume, todo);
}

int backtrace_impl(const int32_t *tau, ErrSource src, int K, int L, int S, int B,
                   int16_t *profile, float *cost, const void *workspace, size_t workspace_bytes,
                   void *stream, bool by_itself, Resume resume = Resume{}, Todo todo = Todo{})
{
    if (!tau || !profile || !cost)
        return SPDY_DP_ERR_NULL;
    const Layout lay = make_layout(K, L, S, B, workspace_bytes);
    const int st = validate(lay, workspace);
    if (st != SPDY_DP_OK)
        return st;
    hipStream_t q = static_cast<hipStream_t>(stream);
    const char *ws = static_cast<const char *>(workspace);
    const int32_t *meta = reinterpret_cast<const int32_t *>(ws + lay.meta_off);
    const int32_t *tstar = reinterpret_cast<const int32_t *>(ws + lay.tstar_off);
    (void)hipGetLastError();
    DeviceState dev;
    const int ok = device_state(false, &dev);
    if (ok != SPDY_DP_OK)
        return ok;
    if (lay.variant == kLevelRecord) {
        auto walk = S <= kWave ? dp_backtrace_levels<1, false> : dp_backtrace_levels<4, false>;
        if (by_itself)
            walk = S <= kWave ? dp_backtrace_levels<1, true> : dp_backtrace_levels<4, true>;
        int per_block = kWalkThreads / kWave, threads = kWalkThreads;
        if (K > (long long)(L < kLevelShort ? kLevelWavesShort : kLevelWaves) * dev.units) {
            walk = by_itself ? dp_backtrace_levels_by_lanes<true> : dp_backtrace_levels_by_lanes<false>;
            per_block = threads = kWave;
        }
        hipLaunchKernelGGL(walk, dim3((K + per_block - 1) / per_block), dim3(threads), 0, q,
                           tau, src, meta, reinterpret_cast<const uint8_t *>(ws + lay.record_off),
                           tstar, K, L, S, (int)lay.row, profile, cost, todo);
    } else {
        launch_walk(tau, src, meta, reinterpret_cast<const float *>(ws + lay.record_off), tstar, K,
                    1, L, S, (int)lay.row, profile, cost, resume, todo, by_itself, dev.units, q);
    }
    return launch_status();
}

// What becomes of the workspace of a call.
enum class Use {
    kTable,         // the caller looks at the table
    kScratch,       // nobody does, so the table need not be there; (a short one is: calls may resume from it)
    kUnseen         // the same, and nothing resumes from it
};
int solve_impl(const int32_t *tau, ErrSource src, int K, int L, int S, int B, int16_t *profile,
               float *cost, void *workspace, size_t workspace_bytes, void *stream, Use use,
               Resume resume = Resume{})
{
    if (!tau || !profile || !cost)
        return SPDY_DP_ERR_NULL;
    const bool scratch = use != Use::kTable;
    if (use == Use::kUnseen) {
        const Layout lay = make_layout(K, L, S, B, workspace_bytes);
        const int ok = validate(lay, workspace);
        if (ok != SPDY_DP_OK)
            return ok;
        char *ws = static_cast<char *>(workspace);
        if (small_call(K, L, S, B))
            return launch_small(tau, src, K, L, S, B, profile, cost,
                                reinterpret_cast<int32_t *>(ws + lay.meta_off) + kMetaTable,
                                static_cast<hipStream_t>(stream));
    }
    CoreCall core;
    Todo todo;
    if (scratch && core_call(make_layout(K, L, S, B, workspace_bytes), K, L, S, &B, 1,
                             !resume.first_layer, profile, cost, workspace, workspace_bytes, &core))
        todo = Todo{profile, 1};
    const int st = fill_impl(tau, src, K, L, S, B, cost, workspace, workspace_bytes, stream, resume,
                             todo.profile ? &core : nullptr);
    if (st != SPDY_DP_OK || (todo.profile && core.rest))
        return st;
    return backtrace_impl(tau, src, K, L, S, B, profile, cost, workspace, workspace_bytes, stream,
                          false, resume, todo);
}

// The stride of the solve with checkpoints: the caller's, or about sqrt(L), which makes the
// checkpoints and the block record the same size.
int checkpoint_stride(int L, int stride)
{
    if (stride > 0)
        return stride < L ? stride : L;
    int j = 1;
    while ((long long)j * j < L)
        ++j;
    return j;
}

// Pass 0 over all layers (checkpoints, final time), then per block of `stride` layers, last
// first: fill the block's rows from the checkpoint below it and walk through them.
int checkpointed_impl(const int32_t *tau, ErrSource src, int K, int L, int S, int B, int stride,
                      int16_t *profile, float *cost, void *workspace, size_t workspace_bytes,
                      void *stream)
{
    if (!tau || !profile || !cost)
        return SPDY_DP_ERR_NULL;
    if (L <= 0)
        return SPDY_DP_ERR_DIM;
    const int j = checkpoint_stride(L, stride);
    const int nblocks = (L + j - 1) / j;
    const int slots = nblocks - 1;
    const Layout lay = make_layout(K, L, S, B, workspace_bytes, (long long)slots + j);
    int st = validate(lay, workspace);
    if (st != SPDY_DP_OK)
        return st;
    if (lay.variant != kValueRecord)
        return SPDY_DP_ERR_WORKSPACE;
    hipStream_t q = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace);
    (void)hipGetLastError();
    Blocks blocks{};
    blocks.stride = j;
    blocks.slots = slots;
    blocks.ckpt = reinterpret_cast<float *>(ws + lay.record_off);
    blocks.block = blocks.ckpt + (size_t)K * slots * lay.row;
    CoreCall core;
    const bool reduced =
        core_call(lay, K, L, S, &B, 1, false, profile, cost, workspace, workspace_bytes, &core);
    auto fill = [&]() {
        const CoreCall *first = reduced ? &core : nullptr;
        return S <= kWave
                   ? launch_fill<false, true, true>(lay, tau, src, Resume{}, K, L, S, B, ws, cost,
                                                    q, blocks, first)
                   : launch_fill<false, false, true>(lay, tau, src, Resume{}, K, L, S, B, ws, cost,
                                                     q, blocks, first);
    };
    blocks.pass = 0;
    blocks.begin = 0;
    blocks.end = L;
    st = fill();
    if (st != SPDY_DP_OK || reduced)
        return st;                                // (dp_rest does all passes)
    const int32_t *meta = reinterpret_cast<const int32_t *>(ws + lay.meta_off);
    int32_t *tstar = reinterpret_cast<int32_t *>(ws + lay.tstar_off);
    const int per_block = kWalkThreads / kWave;
    blocks.pass = 1;
    for (int b = nblocks - 1; b >= 0; --b) {
        blocks.begin = b * j;
        blocks.end = (b + 1) * j < L ? (b + 1) * j : L;
        st = fill();
        if (st != SPDY_DP_OK)
            return st;
        auto walk = S <= kWave ? dp_backtrace_blocks<1> : dp_backtrace_blocks<4>;
        hipLaunchKernelGGL(walk, dim3((K + per_block - 1) / per_block), dim3(kWalkThreads), 0, q,
                           tau, src, meta, tstar, K, L, S, (int)lay.row, profile, cost, blocks);
        st = launch_status();
        if (st != SPDY_DP_OK)
            return st;
    }
    return SPDY_DP_OK;
}

int budgets_impl(const int32_t *tau, ErrSource src, int K, int L, int S, const int32_t *budgets,
                 int J, int16_t *profile, float *cost, void *workspace, size_t workspace_bytes,
                 void *stream)
{
    if (!tau || !budgets || !profile || !cost)
        return SPDY_DP_ERR_NULL;
    if (J <= 0)
        return SPDY_DP_ERR_DIM;
    int bmax = budgets[0];
    for (int j = 0; j < J; ++j) {
        if (budgets[j] < 0)
            return SPDY_DP_ERR_DIM;
        bmax = budgets[j] > bmax ? budgets[j] : bmax;
    }
    const Layout lay = make_layout(K, L, S, bmax, workspace_bytes);
    int st = validate(lay, workspace);
    if (st != SPDY_DP_OK)
        return st;
    if (lay.variant != kValueRecord)
        return SPDY_DP_ERR_WORKSPACE;            // the last row of D is only kept in the D record
    char *ws = static_cast<char *>(workspace);
    const int32_t *meta = reinterpret_cast<const int32_t *>(ws + lay.meta_off);
    const float *drec = reinterpret_cast<const float *>(ws + lay.record_off);
    CoreCall core;
    Todo todo;
    const bool reduced = core_call(lay, K, L, S, budgets, J, J == 1, profile, cost, workspace,
                                   workspace_bytes, &core);
    if (reduced)
        todo = Todo{profile, 1};
    DeviceState dev;
    st = device_state(false, &dev);
    if (st != SPDY_DP_OK)
        return st;
    // one fill for the largest budget; its own costs are not used, and behind the reduced problem
    // they are not written (cost[0..K) holds what that found under the first budget)
    st = fill_impl(tau, src, K, L, S, bmax, reduced ? nullptr : cost, workspace, workspace_bytes,
                   stream, Resume{}, reduced ? &core : nullptr);
    if (st != SPDY_DP_OK)
        return st;
    hipStream_t q = static_cast<hipStream_t>(stream);
    const int most = budgets_per_launch(K, L);
    for (int j0 = reduced && core.walks ? J : 0; j0 < J; j0 += most) {
        const int n = J - j0 < most ? J - j0 : most;
        Budgets some{};
        for (int j = 0; j < n; ++j)
            some.at[j] = budgets[j0 + j];
        int16_t *prof = profile + (size_t)j0 * K * L;
        float *c = cost + (size_t)j0 * K;
        if (reduced)
            todo.profile = prof;
        // the times travel in the words of the costs
        hipLaunchKernelGGL(dp_budget_argmin, dim3(K * n), dim3(256), 0, q, meta, drec, K, L,
                           (int)lay.row, some, reinterpret_cast<int32_t *>(c), todo);
        launch_walk(tau, src, meta, drec, reinterpret_cast<const int32_t *>(c), K, n, L, S,
                    (int)lay.row, prof, c, Resume{}, todo, false, dev.units, q);
    }
    return launch_status();
}

int resume_impl(const int32_t *tau, ErrSource src, const int32_t *first_layer, int K, int L, int S,
                int B, const void *incumbent, size_t incumbent_bytes, int16_t *profile,
                float *cost, void *workspace, size_t workspace_bytes, void *stream)
{
    if (!tau || !first_layer || !incumbent || !profile || !cost)
        return SPDY_DP_ERR_NULL;
    const Layout lay = make_layout(K, L, S, B, workspace_bytes);
    int st = validate(lay, workspace);
    if (st != SPDY_DP_OK)
        return st;
    const Layout inc = make_layout(1, L, S, B, incumbent_bytes);
    if (inc.status != SPDY_DP_OK)
        return inc.status;
    if (lay.variant != kValueRecord || inc.variant != kValueRecord)
        return SPDY_DP_ERR_WORKSPACE;            // rows of D are only kept in the D record
    const char *a = static_cast<const char *>(incumbent);
    const char *b = static_cast<const char *>(workspace);
    if (a < b + workspace_bytes && b < a + incumbent_bytes)
        return SPDY_DP_ERR_WORKSPACE;            // the fill would overwrite the rows it resumes from
    Resume resume;
    resume.first_layer = first_layer;
    resume.inc_rec =
        reinterpret_cast<const float *>(static_cast<const char *>(incumbent) + inc.record_off);
    resume.inc_meta =
        reinterpret_cast<const int32_t *>(static_cast<const char *>(incumbent) + inc.meta_off);
    return solve_impl(tau, src, K, L, S, B, profile, cost, workspace, workspace_bytes, stream,
                      Use::kScratch, resume);
}

}  // namespace

extern "C" {

size_t spdy_dp_workspace_bytes(int K, int L, int S, int B)
{
    const Layout lay = make_layout(K, L, S, B, SIZE_MAX);
    return lay.status == SPDY_DP_OK ? lay.total_value : 0;
}

size_t spdy_dp_workspace_bytes_min(int K, int L, int S, int B)
{
    const Layout lay = make_layout(K, L, S, B, SIZE_MAX);
    return lay.status == SPDY_DP_OK ? lay.total_level : 0;
}

int spdy_dp_workspace_layout(int K, int L, int S, int B, size_t workspace_bytes, size_t out[8])
{
    if (!out)
        return SPDY_DP_ERR_NULL;
    const Layout lay = make_layout(K, L, S, B, workspace_bytes);
    if (lay.status != SPDY_DP_OK)
        return lay.status;
    out[0] = (size_t)lay.variant;
    out[1] = lay.meta_off;
    out[2] = lay.tstar_off;
    out[3] = lay.record_off;
    out[4] = lay.row;
    out[5] = (size_t)L;
    out[6] = (size_t)kMetaHeader;
    out[7] = (size_t)kRangeStride;
    return SPDY_DP_OK;
}

int spdy_dp_fill(const int32_t *tau, const float *err, int K, int L, int S, int B, float *cost,
                 void *workspace, size_t workspace_bytes, void *stream)
{
    if (!err)
        return SPDY_DP_ERR_NULL;
    return fill_impl(tau, ErrSource{err, nullptr, nullptr}, K, L, S, B, cost, workspace,
                     workspace_bytes, stream);
}

int spdy_dp_backtrace(const int32_t *tau, const float *err, int K, int L, int S, int B,
                      int16_t *profile, float *cost, const void *workspace,
                      size_t workspace_bytes, void *stream)
{
    if (!err)
        return SPDY_DP_ERR_NULL;
    return backtrace_impl(tau, ErrSource{err, nullptr, nullptr}, K, L, S, B, profile, cost,
                          workspace, workspace_bytes, stream, true);
}

int spdy_dp_solve_batched(const int32_t *tau, const float *err, int K, int L, int S, int B,
                          int16_t *profile, float *cost, void *workspace, size_t workspace_bytes,
                          void *stream)
{
    if (!err)
        return SPDY_DP_ERR_NULL;
    return solve_impl(tau, ErrSource{err, nullptr, nullptr}, K, L, S, B, profile, cost, workspace,
                      workspace_bytes, stream, Use::kTable);
}

int spdy_dp_solve_profiles(const int32_t *tau, const float *err, int K, int L, int S, int B,
                           int16_t *profile, float *cost, void *workspace, size_t workspace_bytes,
                           void *stream)
{
    if (!err)
        return SPDY_DP_ERR_NULL;
    return solve_impl(tau, ErrSource{err, nullptr, nullptr}, K, L, S, B, profile, cost, workspace,
                      workspace_bytes, stream, K > 1 ? Use::kUnseen : Use::kScratch);
}

int spdy_dp_solve_batched_static(const int32_t *tau, const float *err, int K, int L, int S, int B,
                                 int16_t *profile, float *cost, void *stream)
{
    if (!tau || !err || !profile || !cost)
        return SPDY_DP_ERR_NULL;
    // sizes first: nothing is looked up or enqueued for a problem that does not fit
    const Layout lay = make_layout(K, L, S, B, SPDY_DP_STATIC_WORKSPACE_BYTES);
    if (lay.status == SPDY_DP_ERR_WORKSPACE)
        return SPDY_DP_ERR_STATIC_LIMIT;
    if (lay.status != SPDY_DP_OK)
        return lay.status;
    DeviceState dev;
    const int st = device_state(true, &dev);
    if (st != SPDY_DP_OK)
        return st;
    return solve_impl(tau, ErrSource{err, nullptr, nullptr}, K, L, S, B, profile, cost,
                      dev.scratch, SPDY_DP_STATIC_WORKSPACE_BYTES, stream, Use::kUnseen);
}

int spdy_dp_solve_sensitivities(const int32_t *tau, const float *c, const float *w, int K, int L,
                                int S, int B, int16_t *profile, float *cost, void *workspace,
                                size_t workspace_bytes, void *stream)
{
    if (!c || !w)
        return SPDY_DP_ERR_NULL;
    return solve_impl(tau, ErrSource{nullptr, c, w}, K, L, S, B, profile, cost, workspace,
                      workspace_bytes, stream, Use::kScratch);
}

int spdy_dp_solve_budgets(const int32_t *tau, const float *err, int K, int L, int S,
                          const int32_t *budgets, int J, int16_t *profile, float *cost,
                          void *workspace, size_t workspace_bytes, void *stream)
{
    if (!err)
        return SPDY_DP_ERR_NULL;
    return budgets_impl(tau, ErrSource{err, nullptr, nullptr}, K, L, S, budgets, J, profile, cost,
                        workspace, workspace_bytes, stream);
}

int spdy_dp_solve_from_incumbent(const int32_t *tau, const float *err, const int32_t *first_layer,
                                 int K, int L, int S, int B, const void *incumbent_workspace,
                                 size_t incumbent_bytes, int16_t *profile, float *cost,
                                 void *workspace, size_t workspace_bytes, void *stream)
{
    if (!err)
        return SPDY_DP_ERR_NULL;
    return resume_impl(tau, ErrSource{err, nullptr, nullptr}, first_layer, K, L, S, B,
                       incumbent_workspace, incumbent_bytes, profile, cost, workspace,
                       workspace_bytes, stream);
}

size_t spdy_dp_workspace_bytes_checkpointed(int K, int L, int S, int B, int stride)
{
    if (L <= 0)
        return 0;
    const int j = checkpoint_stride(L, stride);
    const Layout lay = make_layout(K, L, S, B, SIZE_MAX, (long long)((L + j - 1) / j - 1) + j);
    return lay.status == SPDY_DP_OK ? lay.total_value : 0;
}

int spdy_dp_solve_checkpointed(const int32_t *tau, const float *err, int K, int L, int S, int B,
                               int stride, int16_t *profile, float *cost, void *workspace,
                               size_t workspace_bytes, void *stream)
{
    if (!err)
        return SPDY_DP_ERR_NULL;
    return checkpointed_impl(tau, ErrSource{err, nullptr, nullptr}, K, L, S, B, stride, profile,
                             cost, workspace, workspace_bytes, stream);
}

const char *spdy_dp_strerror(int status)
{
    switch (status) {
    case SPDY_DP_OK: return "ok";
    case SPDY_DP_ERR_NULL: return "a required pointer is NULL";
    case SPDY_DP_ERR_DIM: return "K, L and S must be positive and B non-negative";
    case SPDY_DP_ERR_LEVELS: return "S exceeds 255 levels (a recorded level is one byte)";
    case SPDY_DP_ERR_WORKSPACE: return "workspace smaller than spdy_dp_workspace_bytes_min()";
    case SPDY_DP_ERR_OVERFLOW: return "problem size overflows the index arithmetic";
    case SPDY_DP_ERR_LAUNCH: return "HIP runtime refused a kernel launch";
    case SPDY_DP_ERR_STATIC_LIMIT:
        return "problem needs more than the built-in workspace of spdy_dp_solve_batched_static";
    default: return "unknown status";
    }
}

}  // extern "C"
