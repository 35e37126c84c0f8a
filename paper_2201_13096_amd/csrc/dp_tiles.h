// The fill of few candidates (and of rows too long for LDS): several workgroups per candidate.
// Included by spdy_dp.hip, inside its namespace.
//
// Cell t of a row needs cells at or below t of the row before it, never above.  So the row is cut into
// tiles, one workgroup each; a tile may be layers behind the tiles below it, but waits for nothing
// else: the workgroups of a candidate are a pipeline with one-way hand-over, without a barrier across
// them.  A tile's part of the row stays in LDS for the whole solve; left of it lies an apron, the cells
// of the tiles below that a layer's shifts reach, which is fetched from the record (where the row
// has to go anyway) while the layer before is swept.  What the tiles below have finished is known
// from a counter each.
//
// D record.  Two kinds of tile:
//   short  Two rows alternate, one barrier per layer.  A wave takes up to kTileChunks chunks of 64
//          buckets, lane = bucket; shifts and errors of the entries come from LDS as they lie there, a
//          few pairs ahead, so that a short sweep is neither a chain of LDS round trips nor
//          spends its instructions on moving entries to scalar registers and sorting out residues.
//          Two waves only store rows, two only fetch aprons: memory takes longer than a layer.
//   long   One row in place, two barriers per layer, 128-bit reads (see sweep_layer; at most 64
//          levels): what a wave sweeps is long, and LDS is short.  The waves that are through first (a
//          SIMD serves its oldest wave first) fetch the apron while the others sweep.
//
// What bounds it: the issue of instructions, one per four clocks and SIMD, and for a few candidates the lag
// of a tile behind the one below (store, counter, load: about one and a half layers).  A candidate of 4955
// reduced buckets and S = 40 takes 8400 clocks a layer in one short tile, 3700 in four, 2900 in eight.  Whole
// solves by one workgroup per candidate and so, us (all other parts the same): K = 1, L = 54, S = 40, B = 10000 216
// and 129; K = 64 221 and 145; K = 128 225 and 171; K = 6, L = 173, S = 35, B = 1500 337 and 271; B = 100000, K = 1
// 1326 and 352, K = 64 1404 and 558, K = 128 1501 and 1046, K = 300 3134 and 2363; S = 100, L = 100, B = 4000, K = 60
// 802 and 223.

constexpr int kTileThreads = kTileWaves * kWave;
constexpr int kTileEarly = 8;        // waves that fetch the apron of a long tile
constexpr int kTileHeld = 4;         // quads of an apron that one of their lanes holds until it may write
constexpr int kTileLds = 160 * 1024 - 1024;
// A budget below which a row of at most 64 levels fits one tile with any shifts: the row, an apron as
// long, and the entries of some layers
constexpr int kTileSure = 19000;
static_assert((2 * (kTileSure + kWave + kTileBuckets) + 16 + kTileLayers * (2 * kWave + 1)) * 4 <=
                  kTileLds && kTileSure + kWave + kTileBuckets <=
                                  kTileWaves * kTileUnits * kTileBuckets, "one long tile");
// the same for more levels: two rows and aprons, short tiles
constexpr int kTileSureWide = 6000;
static_assert((4 * (kTileSureWide + 2 * kWave) + 16 + kTileLayers * (2 * 256 + 1)) * 4 <= kTileLds &&
                  kTileSureWide + 2 * kWave <= (kTileWaves - 2) * kTileChunks * kWave, "one short tile");
constexpr int kTileLone = 8192;      // budget up to which a tile per compute unit is better (see launch_fill)
static_assert(kTileBuckets == kQuadChunk, "the plan counts quad chunks");

// cache policies of buffer instructions: past the caches of an XCD, which the others do not see, and
// streamed
constexpr int kCoherent = 16, kStreamed = 2;
using uint4v = unsigned __attribute__((ext_vector_type(4)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_buffer(float *row, int pitch)
{
    // (rows of the tiles are far shorter than 2^29 buckets)
    return __builtin_amdgcn_make_buffer_rsrc(row, 0, min(pitch, 1 << 29) * 4, 0x20000);
}
__device__ __forceinline__ int load_agent(const int *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void store_agent(int *p, int v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Waits until at most N of this wave's memory operations are outstanding (they end in order).
template <int N> __device__ __forceinline__ void wait_but()
{
    static_assert(N < 64, "six bits");
    __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | (N >> 4) << 14);        // vmcnt(N)
}

// A cost and its time as one word that orders like the pair (the two zeros are equal, the sign of
// one travels in the lowest bit).
__device__ __forceinline__ unsigned long long result_key(float v, int t)
{
    const unsigned bits = __builtin_bit_cast(unsigned, v);
    const unsigned minus_zero = bits == 0x80000000u ? 1u : 0u;
    const unsigned abs_zero = minus_zero ? 0u : bits;
    const unsigned up = (abs_zero >> 31) ? ~abs_zero : (abs_zero | 0x80000000u);
    return (unsigned long long)up << 32 | ((unsigned)t << 1 | minus_zero);
}
__device__ __forceinline__ float result_value(unsigned long long key)
{
    const unsigned up = (unsigned)(key >> 32);
    const unsigned bits = (up >> 31) ? (up & 0x7FFFFFFFu) : ~up;
    return __builtin_bit_cast(float, bits | (unsigned)(key & 1u) << 31);
}

// Short tiles: R chunks of one layer, from the row below (`from`: this lane's bucket of the first chunk
// there) to `to`.  entries: (shift in bytes, error) of two entries each, 4 * trips of them.  What a wave
// waits for is asked for two pairs ahead, and the entries four: with one or two waves on a SIMD nothing
// else hides the way to LDS.
template <int R>
__device__ __forceinline__ void tile_chunks(const float *from, float *to, const int4 *entries,
                                            int trips)
{
    const char *const at = reinterpret_cast<const char *>(from);
    float best[R];
#pragma unroll
    for (int j = 0; j < R; ++j)
        best[j] = __builtin_inff();
    struct Pairs {
        float a[2][R], b[2][R];
    };
    auto ask = [&](Pairs &d, const int4 (&e)[4], int half) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const float *const p0 = reinterpret_cast<const float *>(at - e[2 * half + q].x);
            const float *const p1 = reinterpret_cast<const float *>(at - e[2 * half + q].z);
#pragma unroll
            for (int j = 0; j < R; ++j) {
                d.a[q][j] = p0[j * kWave];
                d.b[q][j] = p1[j * kWave];
            }
        }
    };
    auto fold = [&](const Pairs &d, const int4 (&e)[4], int half) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int j = 0; j < R; ++j)
                vmin3(best[j], d.a[q][j] + __builtin_bit_cast(float, e[2 * half + q].y),
                      d.b[q][j] + __builtin_bit_cast(float, e[2 * half + q].w));
    };
    Pairs d0, d1;
    int4 e[4], f[4];
#pragma unroll
    for (int q = 0; q < 4; ++q)
        e[q] = entries[q];
    ask(d0, e, 0);
    int i = 0;
    auto body = [&](const int4 (&now)[4], int4 (&next)[4]) __attribute__((always_inline)) {
        entries += i + 1 < trips ? 4 : 0;         // (the last ones once more at the end)
        ask(d1, now, 1);
#pragma unroll
        for (int q = 0; q < 4; ++q)
            next[q] = entries[q];
        __builtin_amdgcn_sched_barrier(0);
        fold(d0, now, 0);
        ask(d0, next, 0);
        __builtin_amdgcn_sched_barrier(0);
        fold(d1, now, 1);
        return ++i < trips;
    };
    while (body(e, f) && body(f, e)) {
    }
#pragma unroll
    for (int j = 0; j < R; ++j)
        to[j * kWave] = best[j];
}

// Long tiles: Q quad chunks of one layer, from the row they are then written to.  `meanwhile` runs
// between the sweep and the barrier behind it, `after` behind that.
template <int Q, class Meanwhile, class After>
__device__ __forceinline__ void tile_units(float *row, int local, int start, LevelEntry first,
                                           const int2 *entries, __amdgpu_buffer_rsrc_t rec, bool coherent, int lane,
                                           Meanwhile meanwhile, After after)
{
    if constexpr (Q == 0) {
        meanwhile();
        __syncthreads();
        after();
    } else {
        float bq[Q][4], none[1];
#pragma unroll
        for (int j = 0; j < Q; ++j)
#pragma unroll
            for (int c = 0; c < 4; ++c)
                bq[j][c] = __builtin_inff();
        const float4v *quads = reinterpret_cast<const float4v *>(row + local) + (lane - 1);
        sweep_layer<Q, 0, false, true, false>(quads, nullptr, entries, first,
                                       start + local + Q * kQuadChunk - 1, 0, bq, none);
        wait_but<0>();                            // the last layer's record is in memory
        meanwhile();
        __syncthreads();
        after();
        if (lane == 0)
            return;
        const int mine = local + 4 * (lane - 1);  // this lane's buckets of the first quad chunk
#pragma unroll
        for (int j = 0; j < Q; ++j)
            *reinterpret_cast<float4v *>(row + mine + j * kQuadChunk) =
                float4v{bq[j][0], bq[j][1], bq[j][2], bq[j][3]};
#pragma unroll
        for (int j = 0; j < Q; ++j) {
            // (the last unit may run past the end of the record's row: not stored there)
            const int at = (start + mine + j * kQuadChunk) * 4;
            const uint4v bits =
                __builtin_bit_cast(uint4v, float4v{bq[j][0], bq[j][1], bq[j][2], bq[j][3]});
            if (coherent)
                __builtin_amdgcn_raw_buffer_store_b128(bits, rec, at, 0, kCoherent);
            else
                __builtin_amdgcn_raw_buffer_store_b128(bits, rec, at, 0, kStreamed);
        }
    }
}

struct TileShared {      // static LDS of the kernel
    unsigned long long key[kTileWaves];
    int ticket;
};

template <bool kLong, int kLds>
__device__ __forceinline__ void fill_tile(const ErrSource src, const int32_t *__restrict__ meta,
                                          const LevelTables tables, int K, int L, int S, int pitch,
                                          float *__restrict__ drec, int32_t *__restrict__ tstar,
                                          float *__restrict__ cost, int *books, float *lds,
                                          TileShared &sh, int k, int p)
{
    const int plan = meta[kMetaTiles];
    const int tiles = plan & 0xFF;
    int tid = threadIdx.x;
    asm("" : "+v"(tid));                         // (nothing of it kept in registers from tile to tile)
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int bp = meta[kMetaBudget];
    if (bp < 0) {                                // even the fastest levels exceed the budget
        if (tid == 0)
            write_result<false>(__builtin_inff(), 0, k, tstar, cost);
        return;
    }
    int *const flags = tile_flags(books, K * tiles) + k * tiles * kTileFlags;
    const int apron = (int)((unsigned)plan >> 12) * 4;
    const bool below_me = p > 0, above_me = p + 1 < tiles;
    const int32_t *nact = meta + kMetaHeader + L;
    const int32_t *spans = meta + kMetaHeader + (2 + (size_t)kRangeStride) * L;
    constexpr int kGrain = kLong ? kQuadChunk : kWave;
    const int units_all = (nact[L - 1] * kWave + kGrain - 1) / kGrain;
    const int tile = (units_all + tiles - 1) / tiles * kGrain, start = p * tile;
    // Short tiles: behind the sweeping waves two that store rows and, where there are tiles below, two
    // that fetch aprons; waves that are left only meet the others at the barriers.
    const int sweepers = kLong ? kTileWaves : min(tile / kWave, kTileWaves - (tiles > 1 ? 4 : 2));
    const int fetchers = sweepers + 2, idlers = fetchers + (below_me ? 2 : 0);
    // LDS: [apron | row] once (long) or twice, then the entries of `room` layers and their counts (a sweep
    // reads two entries too far)
    const int line = apron + tile, lines = kLong ? line : 2 * line;
    float *const row0 = lds + apron, *const row1 = kLong ? row0 : row0 + line;
    const int s8 = tables.s8;
    const int room = min((kLds / (int)sizeof(float) - lines - 4) / (2 * s8 + 1), L);
    int2 *const entries = reinterpret_cast<int2 *>(lds + lines);
    int *const counts = reinterpret_cast<int *>(entries + room * s8);

    // D before the first layer: see dp_fill
    for (int i = tid * 4; i < lines; i += kTileThreads * 4)
        *reinterpret_cast<float4v *>(lds + i) =
            float4v{__builtin_inff(), __builtin_inff(), __builtin_inff(), __builtin_inff()};
    // the first layer whose row reaches this tile
    int l0 = 0;
    if (start > 0) {
        l0 = L;
        for (int base = 0; base < L && l0 == L; base += kWave) {
            const unsigned long long reach =
                __ballot(base + lane < L && nact[min(base + lane, L - 1)] * kWave > start);
            if (reach)
                l0 = base + __builtin_ctzll(reach);
        }
    }
    __syncthreads();
    if (tid == 0 && start <= apron && l0 == 0)
        row0[-start] = -0.0f;

    const ErrSource mine = src.of_candidate(k, L, S);
    float *const rec_k = drec + (size_t)k * L * pitch;
    // The entries of layers [l, l + room): the shift and the smallest error of the levels that share
    // it.  Barriers on both sides.
    auto stage = [&](int l) __attribute__((always_inline)) {
        const int n = min(room, L - l);
        const int32_t *const shifts = tables.shifts + (size_t)l * s8;
        const int32_t *const entry_of = tables.entry + (size_t)l * s8;
        // the first levels are asked for before anything is waited for
        constexpr int kFirst = 2;
        int entry[kFirst];
        float error[kFirst];
        auto level = [&](int i, int &e, float &x) __attribute__((always_inline)) {
            const int layer = i / S, s = i - layer * S;
            e = layer * s8 + entry_of[layer * s8 + s];
            x = mine.layer(l + layer, S).at(s);
        };
        auto merge = [&](int e, float x) __attribute__((always_inline)) {
            __hip_atomic_fetch_min(reinterpret_cast<float *>(&entries[e].y), x, __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_WORKGROUP);
        };
#pragma unroll
        for (int j = 0; j < kFirst; ++j)
            level(min(tid + j * kTileThreads, n * S - 1), entry[j], error[j]);
        for (int i = tid; i < n * s8; i += kTileThreads) {
            const int layer = i / s8, r = i - layer * s8;
            const int shift = shifts[i];
            const int after = r + 1 < s8 ? shifts[i + 1] : INT32_MAX;
            entries[i] = make_int2(shift > bp ? INT32_MAX : shift,
                                   __builtin_bit_cast(int, __builtin_inff()));
            if (shift != INT32_MAX && after == INT32_MAX)
                counts[layer] = r + 1;
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < kFirst; ++j)          // (not the last level once more: atomics on one word
            if (tid + j * kTileThreads < n * S)   // are slow)
                merge(entry[j], error[j]);
        for (int i = tid + kFirst * kTileThreads; i < n * S; i += kTileThreads) {
            int e;
            float x;
            level(i, e, x);
            merge(e, x);
        }
        __syncthreads();
        // shifts in bytes; what is beyond the budget gives +inf (short tiles) or stays out of reach (long
        // ones, whose rows are far shorter than a fourth of that)
        for (int i = tid; i < n * s8; i += kTileThreads) {
            const int2 v = entries[i];
            const int none = kLong ? INT32_MAX : 0;
            const int error = kLong ? v.y : __builtin_bit_cast(int, __builtin_inff());
            entries[i] = v.x == INT32_MAX ? make_int2(none, error) : make_int2(v.x * 4, v.y);
        }
        __syncthreads();
    };

    // The apron for layer l: buckets [lo, start) of row l - 1.  Lane i watches tile p - 1 - i.
    // `which`: of its counters, the one that counts this row.
    int seen = 0, which = 0;
    const int below = max(p - 1 - lane, 0);
    auto watch = [&]() __attribute__((always_inline)) { return load_agent(flags + below * kTileFlags + which); };
    auto behind = [&](int l, int lo, int limit) __attribute__((always_inline)) {
        return __ballot(lane < p && (below + 1) * tile > lo && below * tile < limit && seen < l) != 0;
    };
    auto wait_for = [&](int l, int lo, int limit) __attribute__((always_inline)) {
        while (behind(l, lo, limit))
            seen = watch();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");     // nothing is read before
    };
    auto apron_quad = [&](__amdgpu_buffer_rsrc_t from, int lo, int limit, int i)
        __attribute__((always_inline)) {
        const int b = lo + 4 * i;
        const uint4v v = __builtin_amdgcn_raw_buffer_load_b128(from, b * 4, 0, kCoherent);
        const bool in = b >= 0 && b < limit;      // (beyond what was computed: +inf)
        const float4v f = __builtin_bit_cast(float4v, v);
        const float4v inf = {__builtin_inff(), __builtin_inff(), __builtin_inff(), __builtin_inff()};
        return in ? f : inf;
    };
    // quads first, first + step, ... of it to LDS, four on their way at a time
    auto put_quads = [&](float *row, __amdgpu_buffer_rsrc_t from, int lo, int limit, int first_quad,
                         int step) __attribute__((always_inline)) {
        const int n = (start - lo) / 4;
        for (int i0 = first_quad; i0 < n; i0 += 4 * step) {
            float4v v[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)           // (past the end: the last once more)
                v[j] = apron_quad(from, lo, limit, min(i0 + j * step, n - 1));
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (i0 + j * step < n)
                    *reinterpret_cast<float4v *>(row - (start - lo) + 4 * (i0 + j * step)) = v[j];
        }
    };

    int staged = l0;                              // the layers before it are, or were, staged
    if (l0 < L) {
        stage(l0);
        staged += room;
    }
    if (below_me && l0 > 0 && l0 < L) {
        const int lo = (start - spans[l0] - 4) & ~3, limit = nact[l0 - 1] * kWave;
        which = kLong ? 0 : (l0 - 1) & 1;
        seen = watch();
        wait_for(l0, lo, limit);
        put_quads(l0 & 1 ? row1 : row0, row_buffer(rec_k + (size_t)(l0 - 1) * pitch, pitch), lo,
                  limit, tid, kTileThreads);
    }
    __syncthreads();
    // What this wave does in layer base + i, in lane i: its chunks (units) | the first of them << 4 |
    // trips through the entries << 16
    int base = 0, held_plan = 0;
    auto plan_layers = [&](int l) __attribute__((always_inline)) {
        base = l;
        const int at = min(l + lane, L - 1);
        const int reach = min(nact[at] * kWave - start, tile);
        const int n = (reach + kGrain - 1) / kGrain;
        const int each = n / sweepers, extra = n - each * sweepers;
        const int r = each + (wave < extra ? 1 : 0), first = wave * each + min(wave, extra);
        const int trips = at < staged ? (counts[at - (staged - room)] + 7) / 8 : 0;
        held_plan = r | first << 4 | trips << 16;
    };
    if constexpr (kLong) {
        const bool fetches = below_me && wave < kTileEarly;
        constexpr int kStep = kTileEarly * kWave;
        int active = l0 < L ? nact[l0] : 0, span = l0 + 1 < L ? spans[l0 + 1] : 0;
        for (int l = l0; l < L; ++l) {
            if (l == staged) {
                stage(l);
                staged += room;
            }
            if (l == l0 || l - base == kWave)
                plan_layers(l);
            const int todo = __builtin_amdgcn_readlane(held_plan, l - base);
            const int2 *const own = entries + (l - (staged - room)) * s8;
            LevelEntry first{INT32_MAX, 0.0f};
            if (lane < s8)
                first.shift = own[lane].x >> 2;
            const int limit = active * kWave;
            const int lo = (start - span - 4) & ~3;        // of the next layer's apron
            const bool more = l + 1 < L;
            if (more) {                           // read a layer ahead
                active = nact[l + 1];
                span = spans[min(l + 2, L - 1)];
            }
            const __amdgpu_buffer_rsrc_t rec = row_buffer(rec_k + (size_t)l * pitch, pitch);
            float4v held[kTileHeld];
            auto meanwhile = [&]() __attribute__((always_inline)) {
                if (fetches && more) {
                    wait_for(l + 1, lo, limit);
#pragma unroll
                    for (int j = 0; j < kTileHeld; ++j)
                        if (tid + j * kStep < (start - lo) / 4)
                            held[j] = apron_quad(rec, lo, limit, tid + j * kStep);
                }
            };
            auto after = [&]() __attribute__((always_inline)) {
                if (above_me && l > l0 && tid == kTileThreads - 1)
                    store_agent(flags + p * kTileFlags, l);    // rows up to l - 1 are in memory
                if (fetches && more) {
#pragma unroll
                    for (int j = 0; j < kTileHeld; ++j) {
                        const int i = tid + j * kStep;
                        if (i < (start - lo) / 4)
                            *reinterpret_cast<float4v *>(row0 - (start - lo) + 4 * i) = held[j];
                    }
                    put_quads(row0, rec, lo, limit, tid + kTileHeld * kStep, kStep);
                }
            };
            const int local = (todo >> 4 & 0xFFF) * kQuadChunk;
            switch (todo & 15) {
            case 0: tile_units<0>(row0, local, start, first, own, rec, above_me, lane, meanwhile, after); break;
            case 1: tile_units<1>(row0, local, start, first, own, rec, above_me, lane, meanwhile, after); break;
            case 2: tile_units<2>(row0, local, start, first, own, rec, above_me, lane, meanwhile, after); break;
            case 3: tile_units<3>(row0, local, start, first, own, rec, above_me, lane, meanwhile, after); break;
            case 4: tile_units<4>(row0, local, start, first, own, rec, above_me, lane, meanwhile, after); break;
            case 5: tile_units<5>(row0, local, start, first, own, rec, above_me, lane, meanwhile, after); break;
            case 6: tile_units<6>(row0, local, start, first, own, rec, above_me, lane, meanwhile, after); break;
            }
            __syncthreads();
        }
    } else if (wave < sweepers) {
        const float *prev = (l0 & 1 ? row1 : row0) + lane;
        float *cur = (l0 & 1 ? row0 : row1) + lane;
        const int2 *own = entries;
        for (int l = l0; l < L; ++l) {
            if (l == staged) {
                stage(l);
                staged += room;
                own = entries;
                plan_layers(l);
            } else if (l == l0 || l - base == kWave) {
                plan_layers(l);
            }
            const int todo = __builtin_amdgcn_readlane(held_plan, l - base);
            const int at = (todo >> 4 & 0xFFF) * kWave, trips = todo >> 16;
            const int4 *const pairs = reinterpret_cast<const int4 *>(own);
            switch (todo & 15) {
            case 0: break;
            case 1: tile_chunks<1>(prev + at, cur + at, pairs, trips); break;
            case 2: tile_chunks<2>(prev + at, cur + at, pairs, trips); break;
            case 3: tile_chunks<3>(prev + at, cur + at, pairs, trips); break;
            case 4: tile_chunks<4>(prev + at, cur + at, pairs, trips); break;
            case 5: tile_chunks<5>(prev + at, cur + at, pairs, trips); break;
            case 6: tile_chunks<6>(prev + at, cur + at, pairs, trips); break;
            case 7: tile_chunks<7>(prev + at, cur + at, pairs, trips); break;
            }
            float *const swap = cur;
            cur = const_cast<float *>(prev);
            prev = swap;
            own += s8;
            __syncthreads();
        }
    } else if (wave < fetchers) {
        // Row l goes to the record while layer l + 1 is swept.  With tiles above, the wave that stored it
        // waits until it is there and says so: a layer later would be a layer more that each of them lags.
        const int odd = wave - sweepers;          // of the rows this wave stores
        auto store_row = [&](int l) __attribute__((always_inline)) {
            const __amdgpu_buffer_rsrc_t rec = row_buffer(rec_k + (size_t)l * pitch, pitch);
            const float *const row = l & 1 ? row0 : row1;
            const int n = min(nact[l] * kWave - start, tile) / 4;
            for (int i0 = lane; i0 < n; i0 += 4 * kWave) {
                uint4v v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    v[j] = *reinterpret_cast<const uint4v *>(row + 4 * min(i0 + j * kWave, n - 1));
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const int at = (start + 4 * (i0 + j * kWave)) * 4;
                    if (i0 + j * kWave < n) {
                        if (above_me)
                            __builtin_amdgcn_raw_buffer_store_b128(v[j], rec, at, 0, kCoherent);
                        else
                            __builtin_amdgcn_raw_buffer_store_b128(v[j], rec, at, 0, kStreamed);
                    }
                }
            }
        };
        for (int l = l0; l < L; ++l) {
            if (l == staged) {
                stage(l);
                staged += room;
            }
            if (l > l0 && ((l - 1) & 1) == odd) {
                store_row(l - 1);
                if (above_me) {
                    wait_but<0>();                // (the fence keeps the compiler from moving the stores)
                    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    if (lane == 0)
                        store_agent(flags + p * kTileFlags + odd, l);
                }
            }
            __syncthreads();
        }
        if (l0 < L && ((L - 1) & 1) == odd)
            store_row(L - 1);
    } else if (wave >= idlers) {
        for (int l = l0; l < L; ++l) {
            if (l == staged) {
                stage(l);
                staged += room;
            }
            __syncthreads();
        }
    } else {
        // The aprons of every other layer: asked for a layer ahead where the rows are there by then.
        which = (wave - sweepers) & 1;            // parity of the rows this wave fetches
        float4v held[kTileHeld];
        bool ahead = false;
        for (int l = l0; l < L; ++l) {
            if (l == staged) {
                stage(l);
                staged += room;
            }
            const bool mine_now = (l & 1) == which;
            const int row_l = mine_now ? l : l + 1;          // the row, for the layer above it
            if (row_l + 1 < L) {
                const int lo = (start - spans[row_l + 1] - 4) & ~3, limit = nact[row_l] * kWave;
                const int n = (start - lo) / 4;
                const __amdgpu_buffer_rsrc_t rec =
                    row_buffer(rec_k + (size_t)row_l * pitch, pitch);
                auto fetch = [&]() __attribute__((always_inline)) {
#pragma unroll
                    for (int j = 0; j < kTileHeld; ++j)
                        held[j] = apron_quad(rec, lo, limit, min(lane + j * kWave, n - 1));
                };
                if (mine_now) {
                    if (!ahead) {
                        wait_for(row_l + 1, lo, limit);
                        fetch();
                    }
                    float *const row = l & 1 ? row0 : row1;
#pragma unroll
                    for (int j = 0; j < kTileHeld; ++j)
                        if (lane + j * kWave < n)
                            *reinterpret_cast<float4v *>(row - 4 * (n - lane - j * kWave)) = held[j];
                    put_quads(row, rec, lo, limit, lane + kTileHeld * kWave, kWave);
                } else {
                    seen = watch();
                    ahead = !behind(row_l + 1, lo, limit);
                    if (ahead) {
                        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
                        fetch();
                    }
                }
            }
            __syncthreads();
        }
    }

    // final argmin over t' <= bp, over the tiles of the candidate
    const float *const last = L & 1 ? row1 : row0;
    unsigned long long key = result_key(__builtin_inff(), 0);
    if (l0 < L)
        for (int i = tid; i < min(tile, bp + 1 - start); i += kTileThreads)
            key = Smaller{}(key, result_key(last[i], start + i));
    key = from_lane(wave_scan(key, ~0ull, Smaller{}), kWave - 1);
    wait_but<0>();                                // this wave's record is in memory
    if (lane == 0)
        sh.key[wave] = key;
    __syncthreads();
    if (wave > 0)
        return;
    key = lane < kTileWaves ? sh.key[lane] : ~0ull;
    if (tiles > 1) {
        unsigned long long *const keys =
            reinterpret_cast<unsigned long long *>(books + 2) + (size_t)k * tiles;
        if (above_me) {
            key = from_lane(wave_scan(key, ~0ull, Smaller{}), kWave - 1);
            if (lane == 0) {
                __hip_atomic_store(keys + p, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                wait_but<0>();
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                store_agent(flags + p * kTileFlags + kTileDone, 1);
            }
            return;
        }
        which = kTileDone;
        do
            seen = watch();
        while (__ballot(lane < p && seen == 0));
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        if (lane < p)
            key = Smaller{}(key, __hip_atomic_load(keys + lane, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT));
    }
    key = from_lane(wave_scan(key, ~0ull, Smaller{}), kWave - 1);
    if (lane == 0)
        write_result<false>(result_value(key), (int)((unsigned)key >> 1), k, tstar, cost);
}

// Tiles are taken in the order in which workgroups come for them, so a tile only ever waits for
// tiles that running workgroups have, whatever else runs on the device.  A workgroup takes them until
// none is left.
template <int kLds>
__device__ __forceinline__ void take_tiles(const ErrSource src, const int32_t *__restrict__ meta,
                                           const LevelTables tables, int K, int L, int S, int pitch,
                                           float *__restrict__ drec, int32_t *__restrict__ tstar,
                                           float *__restrict__ cost, int *books, float *lds,
                                           TileShared &sh)
{
    const int plan = meta[kMetaTiles], tiles = plan & 0xFF;
    const int all = K * tiles;                   // (0 where another launch does the work)
    for (int next = blockIdx.x;; next += gridDim.x) {
        if (tiles > 1) {
            if (threadIdx.x == 0)
                sh.ticket =
                    __hip_atomic_fetch_add(books, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            next = __builtin_amdgcn_readfirstlane(sh.ticket);
        }
        if (next >= all)
            return;
        const int k = next / tiles, p = next - k * tiles;
        if (plan & kTileLong)
            fill_tile<true, kLds>(src, meta, tables, K, L, S, pitch, drec, tstar, cost, books, lds, sh,
                                  k, p);
        else
            fill_tile<false, kLds>(src, meta, tables, K, L, S, pitch, drec, tstar, cost, books, lds, sh,
                                   k, p);
    }
}

__global__ __launch_bounds__(kTileThreads, 4) void dp_tiles(
    ErrSource src, const int32_t *__restrict__ meta, LevelTables tables, int K, int L, int S,
    int pitch, float *__restrict__ drec, int32_t *__restrict__ tstar, float *__restrict__ cost,
    int *books)
{
    extern __shared__ __attribute__((aligned(16))) float tile_lds[];
    __shared__ TileShared sh;
    take_tiles<kTileLds>(src, meta, tables, K, L, S, pitch, drec, tstar, cost, books, tile_lds, sh);
}

// Where rows may have to lie in memory: in tiles, or in place in the wide launch (path 3 of dp_fill),
// whichever was planned, in one launch.  (A launch by itself that finds no tiles costs 1.9 us, and 9 - 19
// with a workgroup for every tile there might be: K = 1024, L = 8, S = 16, B = 30000, rows that fit LDS
// after all: 48.9 us, 40.5 with no more workgroups than units, 38.1 in one launch.  Together with path 4
// instead of 3 it takes rows in memory 1.5 % longer.)
template <bool kNarrow>
__global__ __launch_bounds__(kTileThreads, 4) void dp_wide(
    ErrSource src, const int32_t *__restrict__ meta, LevelTables tables, int units, int K, int L,
    int S, int pitch, float *__restrict__ drec, int32_t *__restrict__ tstar,
    float *__restrict__ cost, Resume resume, int *books)
{
    extern __shared__ __attribute__((aligned(16))) float lds[];
    __shared__ union {
        FillShared fill;
        TileShared tile;
    } sh;
    if (meta[kMetaTiles] > 0)
        take_tiles<kLdsBytes>(src, meta, tables, K, L, S, pitch, drec, tstar, cost, books, lds, sh.tile);
    else
        fill_candidates<false, 3, kNarrow, false, false, false, false, false>(
            src, meta, tables, units, K, L, S, pitch, nullptr, drec, nullptr, tstar, cost, resume,
            Blocks{}, Todo{}, lds, sh.fill);
}
