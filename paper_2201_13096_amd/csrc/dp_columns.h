// The fill of rows that stay in LDS and are updated in place, where quads of buckets do not serve: the level record,
// whose ties go by level index, and the D record of more than 64 levels.  More candidates than compute units.
// Included by spdy_dp.hip, inside its namespace.
//
// Columns.  Aligned 128-bit LDS reads move twice the bytes per clock of narrower ones, and a shift is any
// number of buckets.  So the row is folded into four: it is cut into four parts of W buckets, and position i
// holds the buckets i, i + W, i + 2 W and i + 3 W side by side.  A lane owns a position, four buckets that lie W
// apart, and what it needs for a shift s is position i - s: the same four parts, an aligned read whatever s is.
// Left of position 0 lies a ghost, positions -G .. -1, a copy of the last G positions moved by a part (bucket
// i + c W is component c of position i, and c + 1 of position i - W): a wave whose G positions or fewer all
// come to lie left of -G reads W further up instead, k times over, and takes component c - k for its own c (an
// entry that is so far away does not reach its lowest k parts at all).  k is the same for all positions of a
// wave, so it is a matter of which registers are added, and entries are swept in runs of equal k, in any order.
// A row that grows from layer to layer, as the first ones of a network do, is folded anew where W changes, chunk
// by chunk, behind the barrier that ends the sweep.  Short rows, whose waves would have hardly a position each,
// are not folded (a position is one bucket then, and not four): lane = bucket, 32-bit reads.
//
// What bounds it: the level record issues vector instructions (add, min3, compare, select: 16 clocks of a SIMD for two
// updates of 64 cells), the D record of many levels waits for LDS reads.  Loops of the rate probe (sweep_folded_levels,
// sweep_folded), updates per clock and compute unit: level record 27.3, 24.0 a bucket to a lane; D record 48.4, 27.6.
// Counted: level record, K = 1001, L = 52, S = 42, B = 9973: a SIMD issues 5.6e5 vector instructions, at 3.2 clocks each
// three quarters of the launch; waves wait for half of their time, barriers included, 0.04 of it for LDS, whose conflicts
// are 0.11 of its active clocks; D record, S = 128, K = 1024, L = 54, B = 10^4: LDS is active for three quarters of the
// launch, waves wait for 0.28 of their time, most of it for LDS.
// us a fill by dp_fill, a bucket to a lane, and so: level record, K = 1001, L = 52, S = 42, B = 9973 1263 and 1025; S = 128,
// K = 1024, L = 54, B = 10^4 2462 and 1950; D record of the same 1226 and 766; S = 100, K = 4000, B = 1000 1108 and
// 353.
// Not for D records of at most 64 levels: K = 1024, S = 40, B = 10^4 393 us against 392 by quads of consecutive
// buckets, parameters as cost 545 against 532.  Both are bound by LDS reads there.

// The tables of one layer that a producer holds while it is swept: lane r of block b, entry (D record) or level
// 64 b + r.
template <int kBlocks> struct ColumnFetch {
    int32_t shift[kBlocks], entry[kBlocks];
    float raw[kBlocks];
    // (see Pending)
    __device__ __forceinline__ void settle() const
    {
#pragma unroll
        for (int b = 0; b < kBlocks; ++b)
            asm volatile("" ::"v"(raw[b]), "v"(shift[b]), "v"(entry[b]));
    }
};

// How the row of a layer lies in LDS, in chunks of 64.
struct Fold {
    int width;           // positions (W)
    int ghost;           // (G), the most that a wave has
    int cells;           // buckets that are computed
};

// Where the 64 buckets of a chunk go, which stay together, and their ghost.
__device__ __forceinline__ void put_chunk(float *row, int chunk, int lane, float v, Fold f)
{
    const int c = (chunk >= f.width ? 1 : 0) + (chunk >= 2 * f.width ? 1 : 0) + (chunk >= 3 * f.width ? 1 : 0);
    const int i = chunk - c * f.width;
    float *const at = row + 4 * lane;
    at[4 * kWave * i + c] = v;
    if (c < 3 && i >= f.width - f.ghost)
        at[4 * kWave * (i - f.width) + c + 1] = v;
}

// A position's buckets, and one of them.
template <int C> __device__ __forceinline__ auto cells_at(const char *p, int j)
{
    if constexpr (C == 4)
        return reinterpret_cast<const float4v *>(p)[j * kWave];
    else
        return reinterpret_cast<const float *>(p)[j * kWave];
}
template <class V> __device__ __forceinline__ float cell_of(V v, int c)
{
    if constexpr (std::is_same_v<V, float>)
        return v;
    else
        return v[c];
}

// Two entries that lie as one aligned read.  (Reading an entry is the same for every lane, but as many bytes as
// reading a quad; a pair that begins with an odd one takes two reads of half the rate.)
typedef int AlignedPair __attribute__((ext_vector_type(4)));
__device__ __forceinline__ AlignedPair aligned_pair(const int2 *at)
{
    return *reinterpret_cast<const AlignedPair *>(at);
}

// The least over the entries [begin, end) of what component c - kBack of the position an entry reads gives.
template <int Q, int C, int kBack>
__device__ __forceinline__ void column_values(const char *from, const int2 *entries, int begin, int end,
                                              float (&best)[Q][C])
{
    auto single = [&](int shift, float e) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const auto v = cells_at<C>(from - shift, j);
#pragma unroll
            for (int c = kBack; c < C; ++c)
                vmin(best[j][c], cell_of(v, c - kBack) + e);
        }
    };
    // All quads of a pair are asked for before the first is used: the compiler asks for them one by one otherwise
    // (batches of 1024 with 40 levels swept so: 404 and 393 us).
    auto pair = [&](AlignedPair now) __attribute__((always_inline)) {
        const float e0 = __int_as_float(now.y), e1 = __int_as_float(now.w);
        using Cells = decltype(cells_at<C>(from, 0));
        Cells v0[Q], v1[Q];
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            v0[j] = cells_at<C>(from - now.x, j);
            v1[j] = cells_at<C>(from - now.z, j);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < Q; ++j)
#pragma unroll
            for (int c = kBack; c < C; ++c)
                vmin3(best[j][c], cell_of(v0[j], c - kBack) + e0, cell_of(v1[j], c - kBack) + e1);
    };
    if ((begin & 1) && begin < end) {             // (the other half of its pair is of the run before)
        const int2 one = entries[begin];
        single(one.x, __int_as_float(one.y));
        ++begin;
    }
    const int2 *at = entries + begin;
    int n = end - begin;
    AlignedPair a = aligned_pair(at), b;
    for (; n >= 4; n -= 4) {                      // two a trip, so that none is moved
        b = aligned_pair(at + 2);
        pair(a);
        at += 4;
        a = aligned_pair(at);
        pair(b);
    }
    if (n >= 2) {
        b = aligned_pair(at + 2);
        pair(a);
        a = b;
        n -= 2;
    }
    if (n == 1)
        single(a.x, __int_as_float(a.y));
}

// The same with the levels, n entries from `entries` on.  Two entries in index order share one comparison: where
// the smaller of the two is below what came before, the cell notes the pair, and which of the two it was is found
// out once at the end.  Strict "<" decides; the value is the min either way (the sign of a zero may differ from a
// select's, the walk back re-sums the cost).
template <int Q, int C, int kBack>
__device__ __forceinline__ void column_levels(const char *from, const int2 *entries, const unsigned *words,
                                              int n, float (&best)[Q][C], unsigned (&arg)[Q][C])
{
    auto single = [&](int shift, float e, unsigned word) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const auto v = cells_at<C>(from - shift, j);
#pragma unroll
            for (int c = kBack; c < C; ++c) {
                const float x = cell_of(v, c - kBack) + e;
                arg[j][c] = x < best[j][c] ? word : arg[j][c];
                vmin(best[j][c], x);
            }
        }
    };
    auto pair = [&](EntryPair now, unsigned word) __attribute__((always_inline)) {
        const float e0 = __int_as_float(now.y), e1 = __int_as_float(now.w);
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            const auto v0 = cells_at<C>(from - now.x, j), v1 = cells_at<C>(from - now.z, j);
#pragma unroll
            for (int c = kBack; c < C; ++c) {
                const float m = min3(best[j][c], cell_of(v0, c - kBack) + e0, cell_of(v1, c - kBack) + e1);
                arg[j][c] = m < best[j][c] ? word : arg[j][c];
                best[j][c] = m;
            }
        }
    };
    EntryPair next = entry_pair(entries);
    unsigned word = words[0];
    // two pairs a trip, so that no minimum is moved (the longest shares have no registers for it)
    for (; Q < column_chunks<true>() && n >= 4; n -= 4) {
        const EntryPair a = next, b = entry_pair(entries + 2);
        const unsigned word_a = word, word_b = words[2];
        entries += 4;
        words += 4;
        next = entry_pair(entries);
        word = words[0];
        pair(a, word_a);
        pair(b, word_b);
    }
    for (; n >= 2; n -= 2) {
        const EntryPair a = next;
        const unsigned word_a = word;
        entries += 2;
        words += 2;
        next = entry_pair(entries);
        word = words[0];
        pair(a, word_a);
    }
    if (n == 1)                               // (a pair with itself)
        single(next.x, __int_as_float(next.y), (word & 0xFFFF00FFu) | (word & 0xFFu) << 8);
}

// One wave's share of one layer: Q chunks of 64 positions from chunk `begin` on, C buckets to a position (4, or 1
// where the row is not folded).  Sweep, store the record's row `rec`, meet the others at the barrier behind which
// nobody reads the row any more, write the new row as the next layer wants it.
// `of_lane`: entry `lane`, `blocks`: of 64 entries; `words` (level record): level of an entry, of the one after it << 8, the entry << 16.
template <bool kLevel, int kBlocks, int C, int Q>
__device__ __forceinline__ void fill_share(float *row, Fold now, Fold next, int begin,
                                           int2 of_lane, int blocks, const int2 *entries,
                                           const unsigned *words, void *rec, int lane,
                                           const ColumnFetch<kBlocks> &fetched)
{
    if constexpr (Q == 0) {
        fetched.settle();
        __syncthreads();
    } else {
        float best[Q][C];
        unsigned arg[kLevel ? Q : 1][C];
#pragma unroll
        for (int j = 0; j < Q; ++j)
#pragma unroll
            for (int c = 0; c < C; ++c) {
                best[j][c] = __builtin_inff();
                if constexpr (kLevel)
                    arg[j][c] = kNoLevel | kNoLevel << 8;
            }
        constexpr int kBytes = C * (int)sizeof(float);       // of a position
        const int i0 = begin * kWave;
        const char *const mine = reinterpret_cast<const char *>(row + C * (i0 + lane));
        const int step = now.width * kWave * kBytes;
        // the largest shift that stays above -G with the components where they are, and the largest of all
        const int reach = (i0 + Q * kWave - 1) * kBytes;
        const int near = C == 1 ? reach : (i0 + now.ghost * kWave) * kBytes;
        const int far = C == 1 ? reach : min(near, reach) + 3 * step;
        __builtin_amdgcn_s_waitcnt(0xC07F);       // lgkmcnt(0): see sweep_layer
        auto below = [&](int shift) __attribute__((always_inline)) {
            int n = __builtin_popcountll(__ballot(of_lane.x <= shift));
            for (int b = 1; kBlocks > 1 && b < blocks && n == b * kWave; ++b)
                n += __builtin_popcountll(__ballot(entries[b * kWave + lane].x <= shift));
            return n;
        };
        if constexpr (!kLevel) {
            // by shift: the entries of one k are consecutive
            const int n0 = below(near), n3 = below(far);
            column_values<Q, C, 0>(mine, entries, 0, n0, best);
            if constexpr (C == 4) {
                if (n3 > n0) {
                    const int n1 = min(below(near + step), n3), n2 = min(below(near + 2 * step), n3);
                    column_values<Q, C, 1>(mine + step, entries, n0, n1, best);
                    if (n3 > n1) {
                        column_values<Q, C, 2>(mine + 2 * step, entries, n1, n2, best);
                        column_values<Q, C, 3>(mine + 3 * step, entries, n2, n3, best);
                    }
                }
            }
        } else {
            bool noted = false;
            int2 e = of_lane;
#pragma unroll 1
            for (int b = 0;;) {
                const unsigned long long all = __ballot(e.x <= far), at0 = __ballot(e.x <= near) & all;
                unsigned long long at1 = 0, at2 = 0;
                if constexpr (C == 4) {
                    at1 = __ballot(e.x <= near + step) & all;
                    at2 = __ballot(e.x <= near + 2 * step) & all;
                }
                unsigned long long left = all;
                while (left) {
                    const int i = __builtin_ctzll(left);
                    int n = 0;
                    auto sweep = [&](auto back, unsigned long long these) __attribute__((always_inline)) {
                        const unsigned long long ends = ~(these >> i);     // (the first zero ends the run)
                        n = ends ? min(__builtin_ctzll(ends), kWave - i) : kWave - i;
                        column_levels<Q, C, decltype(back)::value>(
                            mine + decltype(back)::value * step, entries + b * kWave + i,
                            words + b * kWave + i, n, best, arg);
                    };
                    if (C == 1 || (at0 >> i & 1)) {
                        sweep(Many<0>{}, at0);
                    } else if constexpr (C == 4) {
                        if (at1 >> i & 1)
                            sweep(Many<1>{}, at1 & ~at0);
                        else if (at2 >> i & 1)
                            sweep(Many<2>{}, at2 & ~at1);
                        else
                            sweep(Many<3>{}, all & ~at2);
                    }
                    noted |= n > 1;
                    left &= i + n < kWave ? ~0ull << (i + n) : 0;
                }
                if (kBlocks == 1 || ++b >= blocks)
                    break;
                e = entries[b * kWave + lane];
            }
            // The first of a noted pair if it gives the cell's value, otherwise the second (the same level
            // twice where one was noted by itself).
            auto away = [&](int shift) __attribute__((always_inline)) {
                int by = -shift;
                if constexpr (C == 4)
                    by += ((shift > near ? 1 : 0) + (shift > near + step ? 1 : 0) +
                           (shift > near + 2 * step ? 1 : 0)) * (step - (int)sizeof(float));
                return shift <= far ? by : 0;
            };
            const int away_of = kBlocks == 1 ? away(of_lane.x) : 0;
#pragma unroll
            for (int j = 0; noted && j < Q; ++j) {
                __builtin_amdgcn_sched_barrier(0);         // (not all of them at once: registers)
#pragma unroll
                for (int c = 0; c < C; ++c) {
                    int by;
                    float err;
                    if constexpr (kBlocks == 1) {
                        const int i = (int)(arg[j][c] >> 14);          // 4 x the entry, and two bits
                        by = __builtin_amdgcn_ds_bpermute(i, away_of);
                        err = __int_as_float(__builtin_amdgcn_ds_bpermute(i, of_lane.y));
                    } else {
                        const int2 first = entries[arg[j][c] >> 16];
                        by = away(first.x);
                        err = __int_as_float(first.y);
                    }
                    const float v = *reinterpret_cast<const float *>(
                                        mine + by + j * kWave * kBytes + c * (int)sizeof(float)) + err;
                    arg[j][c] = v == best[j][c] ? arg[j][c] : arg[j][c] >> 8;
                }
            }
        }
        fetched.settle();
        // The record.  Levels go by buffer stores, whose bound drops the chunks beyond the computed ones; values are
        // streamed (not read again before the walk back), under a test (buffer stores: 416 us where these
        // take 397, though level bytes so: 1040 and 1065).
        const __amdgpu_buffer_rsrc_t levels =
            __builtin_amdgcn_make_buffer_rsrc(rec, 0, now.cells * kWave, 0x20000);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int chunk = begin + c * now.width;
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                if constexpr (kLevel)
                    __builtin_amdgcn_raw_buffer_store_b8((uint8_t)arg[j][c], levels,
                                                         (chunk + j) * kWave + lane, 0, 0);
                else if (chunk + j < now.cells)
                    __builtin_nontemporal_store(best[j][c],
                                                static_cast<float *>(rec) + (chunk + j) * kWave + lane);
            }
        }
        __syncthreads();
        float *const out = row + C * (i0 + lane);
        if constexpr (C == 1) {
#pragma unroll
            for (int j = 0; j < Q; ++j)
                out[j * kWave] = best[j][0];
        } else if (next.width == now.width) {
#pragma unroll
            for (int j = 0; j < Q; ++j) {
                reinterpret_cast<float4v *>(out)[j * kWave] =
                    float4v{best[j][0], best[j][1], best[j][2], best[j][3]};
                if (begin + j >= now.width - now.ghost)
                    reinterpret_cast<float4v *>(out)[(j - now.width) * kWave] =
                        float4v{__builtin_inff(), best[j][0], best[j][1], best[j][2]};
            }
        } else {
#pragma unroll
            for (int j = 0; j < Q; ++j)
#pragma unroll
                for (int c = 0; c < C; ++c)
                    put_chunk(row, begin + j + c * now.width, lane, best[j][c], next);
        }
    }
}

// The fill (Eq. 2-3 for all L layers) and the final argmin over t: path 1 of fill_candidates, which see, for what
// the head of this file says.  kBlocks: blocks of 64 levels, 1 or 4.
struct ColumnShared {    // static LDS of the kernel
    float best[kFillWaves];
    int time[kFillWaves];
};
static_assert(sizeof(ColumnShared) <= kLdsStatic, "static LDS");
template <bool kLevel, bool kTurns, int kBlocks>
__global__ __launch_bounds__(kFillWaves * kWave, 4) void dp_columns(
    ErrSource src, const int32_t *__restrict__ meta, LevelTables tables, int units, int K, int L, int S,
    int pitch, uint8_t *__restrict__ choice, float *__restrict__ drec, int32_t *__restrict__ tstar,
    float *__restrict__ cost)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ ColumnShared sh;
    // (rows of the level record that this launch is enqueued for are always folded; with a look at the word for
    // them, too, the kernel came out 0.4 % slower: 1036.5 and 1040.3 us a call of the first size above)
    if (meta[kMetaPath] != 1 || (!kLevel && meta[kMetaTiles] >= 0))
        return;                                  // another launch does the work
    const int bp = meta[kMetaBudget];
    const int tid = threadIdx.x;
    if (bp < 0) {                                // even the fastest levels exceed the budget
        if (tid == 0)
            write_result<false>(__builtin_inff(), 0, blockIdx.x, tstar, cost);
        return;
    }
    const int teams = meta[kMetaTeams];
    if ((long long)blockIdx.x * teams >= K)
        return;                                  // the first ceil(K / teams) workgroups suffice
    const bool plain = meta[kMetaTiles] == -1;
    const int32_t *nact = meta + kMetaHeader + L;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int tw = kFillWaves / teams;
    const int team = wave / tw;
    const int wv = wave - team * tw;             // this wave's index in its team
    // Where shares are unequal the larger ones should not be all on one SIMD (wave w of a workgroup runs on SIMD
    // w mod 4): every second group of four waves takes its shares in reverse.
    const bool mirrored = (tw & (tw - 1)) == 0 && ((wave >> 2) & 1);
    const int share = mirrored ? wv ^ (min(tw, 4) - 1) : wv;
    const int k = blockIdx.x * teams + team;
    const bool active = team < teams && k < K;

    // (n * inverse >> 16 is n / tw for what is divided here, less than 2^11 by at most 8)
    const int inverse = (65535 + tw) / tw;
    auto fold = [&](int cells) __attribute__((always_inline)) {
        Fold f;
        f.cells = cells;
        f.width = plain ? cells : (cells + 3) >> 2;
        f.ghost = (f.width + tw - 1) * inverse >> 16;
        return f;
    };
    const Fold last = fold(nact[L - 1]);         // (rows only grow)
    const int row_floats = column_row(last.cells, tw, plain), room = column_entries(S);
    const int team_floats = column_floats(last.cells, tw, plain, S, kLevel);
    float *const base = lds + (size_t)(team < teams ? team : 0) * team_floats;
    float *const row = base + (plain ? last.ghost * kWave : 4 * (last.ghost * kWave + 1));
    int2 *const table = reinterpret_cast<int2 *>(base + row_floats);         // of even layers, of odd ones
    unsigned *const words = reinterpret_cast<unsigned *>(table + 2 * room);

    // D before the first layer: time 0 costs nothing, nothing else is reachable (Eq. 3 then is the general
    // update).  -0.0f + e returns e bit for bit for every e, +0.0f would not for e = -0.0f.  The lowest component of
    // a ghost, aprons and what a layer does not compute keep this +inf.
    for (int i = tid; i < teams * team_floats; i += kFillWaves * kWave)
        lds[i] = __builtin_inff();
    __syncthreads();
    Fold now = fold(nact[0]);
    if (active && wv == 0) {
        const float first = lane == 0 ? -0.0f : __builtin_inff();
        if (plain)
            row[lane] = first;
        else
            put_chunk(row, 0, lane, first, now);
    }

    // this candidate's part of the inputs and of the record
    const size_t ke = active ? k : 0;
    const ErrSource mine = src.of_candidate(ke, L, S);
    uint8_t *const choice_k = kLevel ? choice + ke * L * pitch : nullptr;
    float *const drec_k = kLevel ? nullptr : drec + ke * L * pitch;

    // The first wave of a team prepares the next layer's entries while the others wait for the barrier that ends a
    // layer: shifts and the least errors of what shares one (D record), or the levels worth visiting, in index
    // order.
    const bool producer = share == 0 && team < teams;
    const int s8 = tables.s8;
    // (levels in several blocks of 64 have no registers to wait in during the sweep)
    constexpr bool kFetchAhead = !kLevel || kBlocks == 1;
    ColumnFetch<kBlocks> fetched;
#pragma unroll
    for (int b = 0; b < kBlocks; ++b) {
        fetched.shift[b] = INT32_MAX;
        fetched.entry[b] = 0;
        fetched.raw[b] = __builtin_inff();
    }
    // (Lanes anew in every layer: addresses and masks that stay in registers drive others to scratch memory.)
    auto fetch = [&](int l) __attribute__((always_inline)) {
        int lane = tid & (kWave - 1);
        asm volatile("" : "+v"(lane));
        const LayerTable tl = tables.layer(l);
        const ErrRow er = mine.layer(l, S);
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            const int r = b * kWave + lane;
            fetched.shift[b] = r < s8 ? tl.shift[r] : INT32_MAX;
            fetched.raw[b] = r < S ? er.at(r) : __builtin_inff();
            if (!kLevel && r < S)
                fetched.entry[b] = tl.entry[r];
        }
    };
    auto publish = [&](int l) __attribute__((always_inline)) {
        int lane = tid & (kWave - 1);
        asm volatile("" : "+v"(lane));
        int2 *const to = table + (l & 1) * room;
        constexpr float kNone = __builtin_inff();
        int count = 0;
#pragma unroll
        for (int b = 0; b < kBlocks; ++b) {
            if (b * kWave >= S)
                break;
            const int s = b * kWave + lane;
            const int bytes = fetched.shift[b] > bp ? INT32_MAX
                                                    : fetched.shift[b] * (plain ? 1 : 4) * (int)sizeof(float);
            if constexpr (kLevel) {
                unsigned long long visit = S - b * kWave < kWave ? (1ull << (S - b * kWave)) - 1 : ~0ull;
                if (b == 0)
                    visit &= levels_to_visit(LevelFetch{fetched.shift[0], fetched.raw[0], 0},
                                             load_twins(tables.layer(l)), lane);
                // (all levels of the later blocks are visited)
                const unsigned long long above = visit & ~((2ull << lane) - 1);
                const int at = count + __builtin_amdgcn_mbcnt_hi(
                                           (unsigned)(visit >> 32),
                                           __builtin_amdgcn_mbcnt_lo((unsigned)visit, 0));
                if (visit >> lane & 1) {
                    to[at] = make_int2(bytes, __float_as_int(fetched.raw[b]));
                    words[(l & 1) * room + at] =
                        s |
                        ((above ? b * kWave + __builtin_ctzll(above) : (b + 1) * kWave) & 0xFF) << 8 |
                        at << 16;
                }
                count += __builtin_popcountll(visit);
            } else {
                to[s] = make_int2(bytes, __float_as_int(kNone));
            }
        }
        if constexpr (kLevel) {
            for (int r = count + lane; r < room - kLookAhead; r += kWave)
                to[r] = make_int2(INT32_MAX, __float_as_int(kNone));
        } else {
#pragma unroll
            for (int b = 0; b < kBlocks; ++b)
                if (b * kWave + lane < S)
                    __hip_atomic_fetch_min(reinterpret_cast<float *>(&to[fetched.entry[b]].y), fetched.raw[b],
                                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
    };
    if (producer) {
        fetch(0);
        publish(0);
    }
    __syncthreads();
    fetched.settle();                            // no load is in flight at the loop's head

    // Turns at the instruction priority: see fill_candidates.
    const unsigned turn = ((unsigned)blockIdx.x / (unsigned)units) & 1u;
    const int nwg = (K + teams - 1) / teams;
    const bool take_turns = kTurns && nwg > units && (long long)blockIdx.x + 2 * units >= nwg;
    unsigned long long clock = take_turns ? wall_clock64() : 0;
    int cells_next = nact[min(1, L - 1)];
    for (int l = 0; l < L; ++l) {
        if constexpr (kTurns) {
            if (take_turns) {
                if ((turn ^ (unsigned)(clock >> kPriorityTurn)) & 1u)
                    __builtin_amdgcn_s_setprio(1);
                else
                    __builtin_amdgcn_s_setprio(0);
                clock = wall_clock64();          // read now, looked at a layer later: no wait
            }
        }
        // (addresses of a lane that stayed in registers over all layers drove others to scratch memory)
        int here = lane;
        asm("" : "+v"(here));
        const int2 *const entries = table + (l & 1) * room;
        const int2 of_lane = entries[here];
        if (kFetchAhead && producer && l + 1 < L)
            fetch(l + 1);
        const Fold next = l + 1 < L ? fold(cells_next) : now;
        cells_next = nact[min(l + 2, L - 1)];    // (read a layer ahead)
        int begin = 0, n = 0;                    // this wave's chunks of positions
        if (active) {
            begin = share * now.width * inverse >> 16;
            n = ((share + 1) * now.width * inverse >> 16) - begin;
        }
        void *const rec = kLevel ? (void *)(choice_k + (size_t)l * pitch) : (void *)(drec_k + (size_t)l * pitch);
        auto take = [&](auto cells, auto chunks) __attribute__((always_inline)) {
            fill_share<kLevel, kBlocks, decltype(cells)::value, decltype(chunks)::value>(
                row, now, next, begin, of_lane, (S + kWave - 1) / kWave, entries, words + (l & 1) * room, rec, here,
                kFetchAhead ? fetched : ColumnFetch<kBlocks>{});
        };
        if (plain) {
            switch (n) {
            case 0: take(Many<1>{}, Many<0>{}); break;
            case 1: take(Many<1>{}, Many<1>{}); break;
            case 2: take(Many<1>{}, Many<2>{}); break;
            case 3: take(Many<1>{}, Many<3>{}); break;
            case 4: take(Many<1>{}, Many<4>{}); break;
            case 5: take(Many<1>{}, Many<5>{}); break;
            case 6: take(Many<1>{}, Many<6>{}); break;
            }
            static_assert(kPlainChunks == 6, "a case for each");
        } else {
            switch (n) {
            case 0: take(Many<4>{}, Many<0>{}); break;
            case 1: take(Many<4>{}, Many<1>{}); break;
            case 2: take(Many<4>{}, Many<2>{}); break;
            case 3: take(Many<4>{}, Many<3>{}); break;
            case 4: take(Many<4>{}, Many<4>{}); break;
            case 5: take(Many<4>{}, Many<5>{}); break;
            case 6:
                if constexpr (!kLevel)
                    take(Many<4>{}, Many<6>{});
                break;
            case 7:
                if constexpr (!kLevel)
                    take(Many<4>{}, Many<7>{});
                break;
            }
            static_assert(column_chunks<false>() == 7 && column_chunks<true>() == 5, "a case for each");
            // what the next row has beyond this one
            if (next.width != now.width && active)
                for (int chunk = 4 * now.width + wv; chunk < 4 * next.width; chunk += tw)
                    put_chunk(row, chunk, lane, __builtin_inff(), next);
        }
        if (producer && l + 1 < L) {             // the barrier that ends this layer publishes it
            if constexpr (!kFetchAhead)
                fetch(l + 1);
            publish(l + 1);
        }
        now = next;
        __syncthreads();
    }

    // final argmin over t' <= bp within each team
    float bv = __builtin_inff();
    int bt = INT32_MAX;
    if (active) {
        const int cells = plain ? 1 : 4, width = now.width * kWave;
        for (int i = wv * kWave + lane; i < width; i += tw * kWave)
            for (int c = 0; c < cells; ++c) {
                const int t = i + c * width;
                if (t <= bp)
                    argmin_merge(bv, bt, row[cells * i + c], t);
            }
    }
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const float ov = __shfl_down(bv, off, kWave);
        const int ot = __shfl_down(bt, off, kWave);
        argmin_merge(bv, bt, ov, ot);
    }
    if (lane == 0) {
        sh.best[wave] = bv;
        sh.time[wave] = bt;
    }
    __syncthreads();
    if (active && wv == 0 && lane == 0) {
        for (int w = 1; w < tw; ++w)
            argmin_merge(bv, bt, sh.best[wave + w], sh.time[wave + w]);
        write_result<false>(bv, bt, k, tstar, cost);
    }
}
